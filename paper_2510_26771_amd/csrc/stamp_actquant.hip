// Activation path of the STaMP linear layer on gfx950: T = L X along the tokens (Haar DWT, paper
// section "Efficient Energy Concentration"), per-token scale and rounding to 8- or 4-bit codes
// (Background Eq. 1, in its symmetric absmax form or in full with min-max range and integer offset;
// two-level allocation of section "Optimal bit allocation").  X is read from HBM once and the
// transformed activation never goes to HBM.
//
// Floating-point contract (decides the integer codes, so it is fixed): every coefficient is the
// difference (or sum) of two block sums built by plain pairwise fp32 adds, multiplied once by
// norm(l) = fl(2^(-l/2)); absmax a over the row; scale = a / qmax; inv = qmax / a (IEEE
// divisions); code = rne(fl(T * inv)).  Asymmetric form: hi = max T, nlo = max -T = -min T (the token's own
// range, whether or not it contains 0), range = hi + nlo (a token with max = min: range = |hi|), scale =
// range / qmax, inv = qmax / range with qmax = 2^b - 1, z = rne(fl(nlo * inv)) (any integer), code =
// clamp(rne(fl(T * inv)) + z, 0, qmax), stored as code - 2^(b-1).  This file is compiled with
// -ffp-contract=off.
//
// Kernels (those that leave FP6 operands: stamp_lanes1d.hip, stamp_lanes2d.hip):
//   k_bottom1d / k_bottom2d  one workgroup per (sequence, block of R tokens), all d_in channels;
//                            each thread owns 8 channels for every token of the block, so the
//                            butterflies stay in registers; only the per-row absmax crosses lanes
//                            (DPP inside a wave, per-wave partial maxima in LDS across waves).  Emits the R-1
//                            4-bit rows of the block and the block sum (fp32, to scratch).
//   k_top                    the remaining levels over the k_hi block sums, in LDS, per channel
//                            slice; writes the normalised 8-bit-row coefficients to scratch and
//                            one partial absmax per (row, slice).
//   k_quant_hi               reduces the partial maxima of a row and rounds the row to int8.
#include "stamp_bottom_kernel.h"
#include "stamp_hi6.h"

// one file per block length of the 1-D kernels (split: SplitArgs)
hipError_t stamp_bottom1d_3(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split, hipStream_t st);
hipError_t stamp_bottom1d_4(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split, hipStream_t st);
hipError_t stamp_bottom1d_5(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split, hipStream_t st);
hipError_t stamp_bottom1d_6(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split, hipStream_t st);
hipError_t stamp_bottom1d_7(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split, hipStream_t st);
hipError_t stamp_bottom1d_rag_3(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampHiOut& hi6, hipStream_t st);
hipError_t stamp_bottom1d_rag_4(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampHiOut& hi6, hipStream_t st);
hipError_t stamp_bottom1d_rag_5(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampHiOut& hi6, hipStream_t st);
hipError_t stamp_bottom1d_rag_6(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampHiOut& hi6, hipStream_t st);

namespace {

// ------------------------------------------------------------------------------------------
// Top levels over the k block sums.  Workgroup = (32-channel slice, sequence); the k x 32 slice
// sits in LDS and the butterflies run in place (stride 2^l).  Writes normalised coefficients in
// STaMP order over abot (in place: each workgroup owns its slice) and the row absmax.
// ------------------------------------------------------------------------------------------
constexpr int kTopCh = 32;

// asym: the partial maxima are order keys of max t; those of max -t follow npart words further on.
// L = number of top levels, at least 1 (without any the bottom kernel has finished the block sums).
// The blocks beyond ntop convert the packed 4-bit rows to FP6 operands, a row tile and K step each: neither part fills the
// chip, and neither waits for the other (2048 tokens, 4096 channels, 64 block sums: 7.1 + 7.0 us one after the other, 9.4
// side by side).
__global__ __launch_bounds__(256) void k_top(float* __restrict__ abot, uint32_t* __restrict__ rowmax_part, int k, int d,
                                             int is2d, int G, int r_bottom, int L, int asym, size_t npart, int ntop, int nslices,
                                             const uint8_t* __restrict__ q_lo, uint8_t* __restrict__ a6, int gb) {
  extern __shared__ float s_buf[];  // [k][kTopCh + 1]
  if ((int)blockIdx.x >= ntop) {
#pragma unroll
    for (int i = 0; i < 2; ++i) stamp_gemm::repack6_rows(q_lo, a6, blockIdx.x - ntop, i * 256 + threadIdx.x, gb);
    return;
  }
  const int b = (int)blockIdx.x / nslices, slice = (int)blockIdx.x - b * nslices, c_base = slice * kTopCh, tid = threadIdx.x;
  const int ch = tid & (kTopCh - 1), grp = tid / kTopCh, ngrp = 256 / kTopCh;
  const int stride = kTopCh + 1;
  const bool cact = (c_base + ch) < d;
  float* base = abot + (size_t)b * k * d;
  // four independent loads in flight per thread before the first LDS write (one load per loop trip would
  // pay one memory latency per row)
  for (int j0 = grp; j0 < k; j0 += 4 * ngrp) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u * ngrp;
      v[u] = (cact && j < k) ? base[(size_t)j * d + c_base + ch] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u * ngrp;
      if (j < k) s_buf[j * stride + ch] = v[u];
    }
  }
  __syncthreads();
  if (!is2d) {
    for (int st = 2; st <= (1 << L); st <<= 1) {
      const int npair = k / st;
      for (int i = grp; i < npair; i += ngrp) {
        float* pa = &s_buf[(i * st) * stride + ch];
        float* pd = &s_buf[(i * st + (st >> 1)) * stride + ch];
        const float x0 = *pa, x1 = *pd;
        *pa = __fadd_rn(x0, x1);
        *pd = __fsub_rn(x0, x1);
      }
      __syncthreads();
    }
  } else {
    for (int st = 2; st <= (1 << L); st <<= 1) {
      const int nc = G / st;
      const int h = st >> 1;
      for (int i = grp; i < nc * nc; i += ngrp) {
        const int cy = i / nc, cx = i - cy * nc;
        float* p00 = &s_buf[((cy * st) * G + cx * st) * stride + ch];
        float* p01 = p00 + h * stride;
        float* p10 = p00 + h * G * stride;
        float* p11 = p10 + h * stride;
        const float p = *p00, q = *p01, u = *p10, v = *p11;
        const float t0 = __fadd_rn(p, q), t1 = __fsub_rn(p, q), t2 = __fadd_rn(u, v), t3 = __fsub_rn(u, v);
        *p00 = __fadd_rn(t0, t2);
        *p01 = __fadd_rn(t1, t3);
        *p10 = __fsub_rn(t0, t2);
        *p11 = __fsub_rn(t1, t3);
      }
      __syncthreads();
    }
  }
  // normalise, scatter to STaMP order, row absmax over this slice
  for (int q = grp; q < k; q += ngrp) {
    int e, lvl_top;  // level counted within the top part (1 = first top level); slot 0 gets the deepest
    if (!is2d) {
      e = stamp_top_slot_1d(q, k, L, &lvl_top);
    } else {
      const int y = q / G, x = q - y * G;
      e = stamp_top_slot_2d(y, x, G, L, &lvl_top);
    }
    const int level = r_bottom + lvl_top;
    const float nrm = is2d ? ldexpf(1.0f, -level) : haar_norm(level);
    const float t = __fmul_rn(s_buf[q * stride + ch], nrm);
    if (cact) base[(size_t)e * d + c_base + ch] = t;
    // max over the 32 channels of this row: lanes of one row are 32 consecutive lanes
    auto max32 = [](uint32_t x) {
      uint32_t yv;
      yv = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false); x = max(x, yv);
      yv = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false); x = max(x, yv);
      yv = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false); x = max(x, yv);
      yv = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false); x = max(x, yv);
      yv = (uint32_t)__shfl_xor((int)x, 16, 64); x = max(x, yv);
      return x;
    };
    const size_t slot = ((size_t)b * k + e) * nslices + slice;
    if (!asym) {
      const uint32_t x = max32(absbits(t));
      if (ch == 0) rowmax_part[slot] = x;
    } else {
      // channels beyond d_in contribute the neutral key
      const uint32_t xp = max32(cact ? fkey(t) : 0u);
      const uint32_t xn = max32(cact ? fkey(-t) : 0u);
      if (ch == 0) { rowmax_part[slot] = xp; rowmax_part[npart + slot] = xn; }
    }
  }
}

// one workgroup per 8-bit row.  asym: min-max form, the stored code is code - 128 and the offset z goes
// zeros_off floats behind the row's scale.  hi6.p != nullptr: the rows leave as FP6 operand.
__global__ __launch_bounds__(256) void k_quant_hi(const float* __restrict__ ttop, const uint32_t* __restrict__ rowmax_part,
                                                  int nslices, int8_t* __restrict__ q_hi, float* __restrict__ scales,
                                                  int k, int d, int s, int R, int asym, size_t npart,
                                                  size_t zeros_off, int Kpad, Hi6Out hi6) {
  __shared__ uint32_t s_red[8];
  const int p = blockIdx.x, b = blockIdx.y;
  {
    uint32_t m = 0u, mneg = 0u;
    for (int i = threadIdx.x; i < nslices; i += 256) {
      const size_t slot = ((size_t)b * k + p) * nslices + i;
      m = max(m, rowmax_part[slot]);
      if (asym) mneg = max(mneg, rowmax_part[npart + slot]);
    }
    m = wave_max_u32(m);
    mneg = wave_max_u32(mneg);
    if ((threadIdx.x & 63) == 0) { s_red[threadIdx.x >> 6] = m; s_red[4 + (threadIdx.x >> 6)] = mneg; }
    __syncthreads();
  }
  const uint32_t mp = max(max(s_red[0], s_red[1]), max(s_red[2], s_red[3]));
  const uint32_t mn = max(max(s_red[4], s_red[5]), max(s_red[6], s_red[7]));
  float scale = 0.0f, inv = 0.0f, z = 0.0f;
  if (!asym) {
    const float a = __uint_as_float(mp);
    if (a > 0.0f) {
      scale = __fdiv_rn(a, 127.0f);
      inv = __fdiv_rn(127.0f, a);
    }
  } else {
    asym_params(fkey_inv(mp), fkey_inv(mn), 255.0f, scale, inv, z);
  }
  if (threadIdx.x == 0) {
    scales[(size_t)b * s + (size_t)p * R] = scale;
    if (asym) scales[zeros_off + (size_t)b * s + (size_t)p * R] = z;
  }
  const float qlo = asym ? 0.0f : -127.0f, qhi = asym ? 255.0f : 127.0f, shift = asym ? 128.0f : 0.0f;
  auto code = [&](float v) { return (int)(fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(v, inv)), z), qlo), qhi) - shift); };
  const float* src = ttop + ((size_t)b * k + p) * d;
  if (hi6.p != nullptr) {
    for (int cb = 0; cb < d; cb += 256 * 8) {  // whole quads stay together: d is a multiple of 32
      const int c = cb + (int)threadIdx.x * 8, cl = min(c, d - 8);
      const float4 t0 = *reinterpret_cast<const float4*>(src + cl), t1 = *reinterpret_cast<const float4*>(src + cl + 4);
      const int qi[8] = {code(t0.x), code(t0.y), code(t0.z), code(t0.w), code(t1.x), code(t1.y), code(t1.z), code(t1.w)};
      store_hi48(hi6, b * k + p, Kpad >> 7, qi, c, c < d);
    }
    return;
  }
  int8_t* dst = q_hi + ((size_t)b * k + p) * d;
  for (int c = threadIdx.x * 4; c < d; c += 256 * 4) {
    const float4 t = *reinterpret_cast<const float4*>(src + c);
    *reinterpret_cast<uint32_t*>(dst + c) = ((uint32_t)code(t.x) & 0xFFu) | (((uint32_t)code(t.y) & 0xFFu) << 8) |
                                            (((uint32_t)code(t.z) & 0xFFu) << 16) | ((uint32_t)code(t.w) << 24);
  }
}

// ------------------------------------------------------------------------------------------
// Plans without a sequence transform (the layers the paper leaves un-transformed, and the baseline the
// transform's cost is measured against): per-token quantization of X itself (Background, Eq. 1), tokens
// 0..k-1 of every sequence at 8 bits, the rest at 4 bits.  One workgroup per token: the row is read twice
// (range, then codes; the second read comes from cache).
// OUT6: q_lo is the FP6 operand of the 4-bit rows, the 8-bit rows go to hi6; for few rows, see launch_quant_rows.
// ------------------------------------------------------------------------------------------
template <bool BF16, bool ASYM, bool OUT6>
__global__ __launch_bounds__(256) void k_quant_rows(const void* __restrict__ X, int8_t* __restrict__ q_hi,
                                                    uint8_t* __restrict__ q_lo, float* __restrict__ scales, int s, int d,
                                                    int k, int Kpad, size_t zeros_off, Hi6Out hi6) {
  __shared__ uint32_t s_red[8];
  const int pr = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const size_t m = (size_t)b * s + pr;
  const size_t xoff = m * (size_t)d;
  uint32_t mpos = 0u, mneg = 0u;
  for (int c = tid * 8; c < d; c += 256 * 8) {
    float v[8];
    load8(X, xoff + c, BF16, true, v);
    if constexpr (ASYM) {
      uint32_t pos, neg;
      row_posneg_bits(v, pos, neg);
      mpos = max(mpos, pos);
      mneg = max(mneg, neg);
    } else {
      mpos = max(mpos, row_absmax_bits(v));
    }
  }
  mpos = wave_max_u32(mpos);
  mneg = wave_max_u32(mneg);
  if ((tid & 63) == 0) { s_red[tid >> 6] = mpos; s_red[4 + (tid >> 6)] = mneg; }
  __syncthreads();
  const uint32_t mp = max(max(s_red[0], s_red[1]), max(s_red[2], s_red[3]));
  const uint32_t mn = max(max(s_red[4], s_red[5]), max(s_red[6], s_red[7]));
  const bool hi = pr < k;
  const float qmax = ASYM ? (hi ? 255.0f : 15.0f) : (hi ? 127.0f : 7.0f);
  float scale = 0.0f, inv = 0.0f, z = 0.0f;
  if constexpr (ASYM) {
    asym_params(fkey_inv(mp), fkey_inv(mn), qmax, scale, inv, z);
  } else {
    const float a = __uint_as_float(mp);
    if (a > 0.0f) {
      scale = __fdiv_rn(a, qmax);
      inv = __fdiv_rn(qmax, a);
    }
  }
  if (tid == 0) {
    scales[m] = scale;
    if constexpr (ASYM) scales[zeros_off + m] = z;
  }
  // OUT6: whole quads of threads stay together (a loop that every thread leaves at the same time costs narrow rows in
  // packed form 15 us in 75: 7 x 16384 tokens x 32, fp32)
  for (int c = tid * 8; (OUT6 ? c - tid * 8 : c) < d; c += 256 * 8) {
    float v[8];
    load8(X, xoff + (OUT6 ? min(c, d - 8) : c), BF16, true, v);
    if (hi) {
      const float qlo = ASYM ? 0.0f : -127.0f, qhi = ASYM ? 255.0f : 127.0f, shift = ASYM ? 128.0f : 0.0f;
      uint32_t w[2] = {0u, 0u};
      int qi[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float q = __fadd_rn(rintf(__fmul_rn(v[i], inv)), z);
        q = fminf(fmaxf(q, qlo), qhi) - shift;
        qi[i] = (int)q;
        w[i >> 2] |= ((uint32_t)((int)q) & 0xFFu) << (8 * (i & 3));
      }
      if constexpr (OUT6) store_hi48(hi6, b * k + pr, Kpad >> 7, qi, c, c < d);
      else *reinterpret_cast<uint2*>(q_hi + ((size_t)b * k + pr) * d + c) = make_uint2(w[0], w[1]);
    } else {
      float pq[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pq[i] = __fmul_rn(v[i], inv);
      uint32_t w;
      if constexpr (ASYM) {
        const float lo = -z, hib = 15.0f - z;
#pragma unroll
        for (int i = 0; i < 8; ++i) pq[i] = __builtin_amdgcn_fmed3f(pq[i], lo, hib);
        w = pack8_uint4(pq, z);
      } else {
        w = pack8_int4(pq);
      }
      if constexpr (OUT6) {
        uint32_t w0, w1;
        nib8_to_48(w, w0, w1);
        store48(q_lo + a6_row(m, Kpad >> 7, 2) + off48(c, kStageA6), row_half6((uint32_t)m, 2), w0, w1, c, c < d);
      } else {
        *reinterpret_cast<uint32_t*>(q_lo + stamp_qlo_offset(m, c, Kpad)) = w;
      }
    }
  }
}

}  // namespace

namespace {
Hi6Out hi6_out(const StampDirect* dir) { return dir != nullptr ? dir->hi : Hi6Out{}; }
// FP6 operands of few rows: 8 channels a thread.  A lane of k_lanes_rows has 32 to go through, one after the other, while most CUs
// have no row at all.  One 8-bit row, layers to 256 outputs, us in a graph, k_lanes_rows against this: WHT 16 x 256 23.1, 22.9, 64 x 2048 29.7,
// 29.2, 128 x 1024 28.9, 28.7; rows without transform, fp32 16 x 512 13.6, 13.4, 256 x 1024 17.7, 17.6; from one row per CU on, and where
// a row is several passes of a workgroup, the other way (mean over the depths up to 4096: 512 rows 0.2 us, 1024 rows 1.0; bf16
// rows of 4096 0.5, of 11008 2.4).
template <bool BF16, bool ASYM>
hipError_t launch_quant_rows(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampDirect* dir, hipStream_t st) {
  const StampGeom& g = p->geom;
  const size_t zoff = (size_t)g.B * g.s;
  const dim3 grid(g.s, g.B), blk(256);
  if (dir == nullptr)
    hipLaunchKernelGGL((k_quant_rows<BF16, ASYM, false>), grid, blk, 0, st, X, q_hi, q_lo, scales, g.s, g.d, g.k, p->Kpad, zoff, Hi6Out{});
  else if ((int64_t)g.B * g.s <= stamp_device_cus() && g.d <= (BF16 ? 2048 : 4096))
    hipLaunchKernelGGL((k_quant_rows<BF16, ASYM, true>), grid, blk, 0, st, X, q_hi, dir->a6, scales, g.s, g.d, g.k, p->Kpad, zoff, dir->hi);
  else
    return stamp_launch_lanes_rows(p, X, BF16, dir->a6, scales, dir->hi, st);
  return hipGetLastError();
}
}  // namespace

// One workgroup has to hold all channels, 16-byte loads of X need its alignment.
bool stamp_rag_quantizes(const stamp_plan* p, const void* X) {
  return p->rag.on && p->geom.d <= (p->geom.x_bf16 ? 8192 : 4096) && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
}

hipError_t stamp_launch_actquant_rag(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, hipStream_t st,
                                     const StampDirect* dir) {
  const Hi6Out hi6 = hi6_out(dir);
  if (dir != nullptr) q_lo = dir->a6;
  if (dir != nullptr && stamp_lanes1d_fits(p, p->rag.r)) return stamp_launch_lanes1d(p, p->rag.r, X, q_lo, scales, nullptr, hi6, st);
  switch (p->rag.r) {
    case 3: return stamp_bottom1d_rag_3(p, X, q_hi, q_lo, scales, hi6, st);
    case 4: return stamp_bottom1d_rag_4(p, X, q_hi, q_lo, scales, hi6, st);
    case 5: return stamp_bottom1d_rag_5(p, X, q_hi, q_lo, scales, hi6, st);
    case 6: return stamp_bottom1d_rag_6(p, X, q_hi, q_lo, scales, hi6, st);
    default: return hipErrorInvalidValue;
  }
}

// general path: per-token quantization of the transformed tokens T [B, s, d] fp32 (rows = STaMP slots)
hipError_t stamp_launch_quant_rows_f32(const stamp_plan* p, const float* T, int8_t* q_hi, uint8_t* q_lo, float* scales,
                                       hipStream_t st, const StampDirect* dir) {
  return p->geom.asym ? launch_quant_rows<false, true>(p, T, q_hi, q_lo, scales, dir, st)
                      : launch_quant_rows<false, false>(p, T, q_hi, q_lo, scales, dir, st);
}

bool stamp_top_in_bottom(const stamp_plan* p) {
  return !p->geom.ident && p->geom.L == 0;
}

bool stamp_bottom_quads(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  return !g.ident && g.is2d && g.r == 3 && g.d <= 1536 && g.B * g.k <= 2 * stamp_device_cus();
}

int stamp_actquant_nsplit(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  if (g.ident) return 1;
  const int dmax = (g.is2d || !g.x_bf16) ? 4096 : 8192;  // channels one workgroup can hold
  return (g.d + dmax - 1) / dmax;
}

hipError_t stamp_launch_actquant(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales,
                                 float* abot, uint32_t* rowmax, uint32_t* gpart, hipStream_t st, int part,
                                 const StampDirect* dir) {
  const StampGeom& g = p->geom;
  if (g.ident) {
    if (!(part & 1)) return hipSuccess;
    if (g.asym)
      return g.x_bf16 ? launch_quant_rows<true, true>(p, X, q_hi, q_lo, scales, dir, st)
                      : launch_quant_rows<false, true>(p, X, q_hi, q_lo, scales, dir, st);
    return g.x_bf16 ? launch_quant_rows<true, false>(p, X, q_hi, q_lo, scales, dir, st)
                    : launch_quant_rows<false, false>(p, X, q_hi, q_lo, scales, dir, st);
  }
  if (dir != nullptr && dir->parts) {
    const hipError_t e = stamp_launch_lanes1d(p, 3, X, dir->a6, scales, abot, StampHiOut{}, st);
    if (e != hipSuccess) return e;
    return stamp_launch_top_parts(p, abot, dir->a6, scales, dir->hi, st);
  }
  SplitArgs sp;
  sp.gpart = gpart;
  sp.part_rows = (size_t)g.B * g.s;
  sp.nsplit = stamp_actquant_nsplit(p);
  sp.c_split = (sp.nsplit == 1) ? g.d : (((g.d + sp.nsplit - 1) / sp.nsplit + 511) / 512) * 512;
  if (sp.nsplit > 1 && gpart == nullptr) return hipErrorInvalidValue;
  // No top levels: the bottom kernel finishes the block sums itself, with split channels too (their maxima travel with the
  // other rows').  Bottom kernel, k_top and k_quant_hi, 256 block sums x 11008 channels: 31.1 + 19.3 + 8.4 us; now 32.7.
  const bool top_in_bottom = stamp_top_in_bottom(p);
  sp.q_hi = top_in_bottom ? q_hi : nullptr;
  sp.khi = g.khi;
  const StampDirect* const bot = dir != nullptr && !dir->lo_packed ? dir : nullptr;  // the bottom kernel stores the operands
  sp.hi6 = hi6_out(bot);
  const bool quads = stamp_bottom_quads(p);
  if (bot != nullptr) {
    if (g.is2d && !stamp_lanes2d_fits(p)) return hipErrorInvalidValue;  // direct_route
    q_lo = dir->a6;
  }
  const int nthreads = ((sp.c_split / 8 + 63) / 64) * 64;
  dim3 grid(g.k, g.B);
  const size_t zeros_off = (size_t)g.B * g.s;
#define LAUNCH1D(RL)                                                                                      \
  do {                                                                                                    \
    const hipError_t le = stamp_bottom1d_##RL(p, X, q_lo, scales, abot, nthreads, &sp, st);               \
    if (le != hipSuccess) return le;                                                                      \
  } while (0)
#define LAUNCH2D__(RL, BF, AS, PASS)                                                                      \
  hipLaunchKernelGGL((k_bottom2d<RL, BF, AS, PASS>), dim3(g.k, g.B, PASS == 0 ? 1 : sp.nsplit), dim3(nthreads), 0, st, X, \
                     q_lo, scales, abot, g.s, g.d, g.G, g.gridW, p->Kpad, zeros_off, sp)
#define LAUNCH2D_(RL, BF, AS)                                                                             \
  do {                                                                                                    \
    if (sp.nsplit == 1) { LAUNCH2D__(RL, BF, AS, 0); }                                                    \
    else { LAUNCH2D__(RL, BF, AS, 1); LAUNCH2D__(RL, BF, AS, 2); }                                        \
  } while (0)
#define LAUNCHQ(BF, AS)                                                                                   \
  hipLaunchKernelGGL((k_bottom2d_quads<BF, AS>), grid, dim3(4 * nthreads), (size_t)4 * nthreads * 32, st, X, q_lo, scales, abot, \
                     g.s, g.d, g.G, g.gridW, p->Kpad, zeros_off, sp)
#define LAUNCH2D(RL)                                                                                      \
  do {                                                                                                    \
    if (g.asym) { if (g.x_bf16) LAUNCH2D_(RL, true, true); else LAUNCH2D_(RL, false, true); }             \
    else { if (g.x_bf16) LAUNCH2D_(RL, true, false); else LAUNCH2D_(RL, false, false); }                  \
  } while (0)
  if (!(part & 1)) {
    // bottom kernel skipped
  } else if (g.is2d && bot != nullptr) {
    const hipError_t le = stamp_launch_lanes2d(p, X, q_lo, scales, top_in_bottom ? nullptr : abot, sp.hi6, st);
    if (le != hipSuccess) return le;
  } else if (!g.is2d && bot != nullptr && stamp_lanes1d_fits(p, g.r)) {
    const hipError_t le = stamp_launch_lanes1d(p, g.r, X, q_lo, scales, top_in_bottom ? nullptr : abot, sp.hi6, st);
    if (le != hipSuccess) return le;
  } else if (!g.is2d) {
    switch (g.r) {
      case 3: LAUNCH1D(3); break;
      case 4: LAUNCH1D(4); break;
      case 5: LAUNCH1D(5); break;
      case 6: LAUNCH1D(6); break;
      case 7: LAUNCH1D(7); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    if (nthreads > 512) return hipErrorInvalidValue;
    if (quads) {
      if (g.asym) { if (g.x_bf16) LAUNCHQ(true, true); else LAUNCHQ(false, true); }
      else { if (g.x_bf16) LAUNCHQ(true, false); else LAUNCHQ(false, false); }
    } else switch (g.r) {
      case 2: LAUNCH2D(2); break;
      case 3: LAUNCH2D(3); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef LAUNCH1D
#undef LAUNCH2D
#undef LAUNCH2D_
#undef LAUNCH2D__
#undef LAUNCHQ
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!(part & 2) || top_in_bottom) return hipSuccess;
  if (g.k > 256) return hipErrorInvalidValue;  // plan creation admits that many top rows only without top levels
  const size_t lds = (size_t)g.k * (kTopCh + 1) * sizeof(float);
  const int nslices = (g.d + kTopCh - 1) / kTopCh;
  const size_t npart = (size_t)g.B * g.k * nslices;
  const int ntop = nslices * g.B, nlo = dir != nullptr && dir->lo_packed ? (p->Mpad / 256) * (p->Kpad / 128) : 0;
  hipLaunchKernelGGL(k_top, dim3(ntop + nlo), dim3(256), lds, st, abot, rowmax, g.k, g.d, g.is2d, g.G, g.r, g.L, g.asym, npart,
                     ntop, nslices, q_lo, dir != nullptr ? dir->a6 : nullptr, stamp_row_group_bit(p));
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_quant_hi, dim3(g.k, g.B), dim3(256), 0, st, abot, rowmax, nslices, q_hi, scales, g.k, g.d, g.s, g.R, g.asym,
                     npart, zeros_off, p->Kpad, hi6_out(dir));
  return hipGetLastError();
}
