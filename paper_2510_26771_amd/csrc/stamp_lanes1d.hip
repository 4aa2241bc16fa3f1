// Bottom kernels that leave FP6 operands: 1-D blocks of 8 and 16 tokens (parts of longer blocks too), rows without
// transform.
//
// v_cvt_scalef32_2xpk16_fp6_f32 rounds 32 floats to E2M3 numbers (with scale 8: to the nearest integers, ties to even, of a
// magnitude up to 15) and packs them: one instruction makes the 24-byte operand fragment of a row's 32 channels, for
// which the streaming kernels (stamp_bottom_kernel.h: 8 channels a thread) spend eight per value.  So a lane holds 32 consecutive
// channels, of two tokens; the block's other tokens are with its neighbours, and levels above the first pass sums from lane
// to lane.  The pair of a level leaves its sum in the lower lane and its difference, a finished coefficient, in the
// upper one: a lane ends with two rows of 32 channels, its tokens' difference and one other.  The rows' maxima meet in one
// exchange and one barrier.
// Same operations on the same values as the streaming kernels, same codes.
// What bounds it: the vector ALU (about 22 instructions per channel and token pair) and the bytes, about alike: 8 x 2048 tokens x
// 4096 channels 34.2 us (5.4 TB/s; streaming 47.0), 2048 x 4096 8.9 us (11.0) of which 5 are the launch and its first loads.
#include "stamp_lanes.h"

namespace {

// RAG: blocks of a 1-D Haar transform of any length (StampRag), one more workgroup for the token left out.
// NG = 2: a lane holds two groups of 32 channels, for layers as wide as a
// model's down-projection.  Beside the first group's row A, which waits in LDS, 36 of the second group's values find no register and go
// through scratch memory (148 bytes a lane; fp32 and bf16 rows beyond the streaming kernels' split, NG = 1, 6 and 4): 2048 x 11008 21.4 us
// for 62 MB (2.9 TB/s).  NANMAX: a NaN is the largest value of a block sum's row.
template <int RLOG, bool BF16, bool ASYM, bool RAG, int NG, bool NANMAX>
__global__ __launch_bounds__(NG == 1 ? 1024 : 768) void k_lanes1d(const LaneArgs a) {
  constexpr int RK = 1 << RLOG, NL = RK / 2, CPR = BF16 ? 4 : 8;  // tokens, lanes per group of channels, 16-byte loads per token
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][RK][16];  // [sign][row][wave]
  extern __shared__ __attribute__((aligned(16))) uint8_t s_row[];     // NG = 2: row A of the first group, [8][threads] 16 bytes
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
  const int tl = lane & (NL - 1), b = blockIdx.y;
  // (NG = 2, one workgroup per CU: no difference)
  const int unit = NG == 2 ? (int)blockIdx.x : unit_of_block<RK>(blockIdx.x, gridDim.x);
  const int parts = RAG ? 1 : a.R >> RLOG, j = unit / parts, part = unit - j * parts;  // block, part of it
  const size_t seq0 = (size_t)b * a.s, row_bytes = (size_t)a.d * (BF16 ? 2 : 4);
  const bool left_out = RAG && j == a.rag.nb;  // the token left out: a row of its own, in the lanes of tl = 0
  const int m = left_out ? 1 : RAG && j == a.rag.nb - 1 ? a.rag.mlast : RK;
  const uint8_t* const X_blk =
      reinterpret_cast<const uint8_t*>(a.X) + (seq0 + (left_out || !RAG ? 0 : a.rag.o) + (left_out ? 0 : (size_t)unit * RK)) * row_bytes;
  int c0[NG];
  u4 raw[NG][2][CPR];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    c0[g] = ((g * nw + wave) * (64 / NL) + lane / NL) * 32;
    // lanes beyond d_in redo the last channels: duplicates cannot change a row maximum, and they store nothing
    const uint32_t off = (uint32_t)(min(c0[g], a.d - 32) * (BF16 ? 2 : 4));
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint32_t trow = (uint32_t)(RAG ? min(2 * tl + t, m - 1) : 2 * tl + t) * (uint32_t)row_bytes;
#pragma unroll
      for (int h = 0; h < CPR; ++h) raw[g][t][h] = *reinterpret_cast<const u4*>(X_blk + (trow + off) + 16 * h);
    }
  }
  // per lane and level: sign of its own sum (+ in the lower lane of a pair), whether the lane takes part, whether its pair is whole
  float sg[RLOG + 1];
  bool in[RLOG + 1], whole[RLOG + 1];
#pragma unroll
  for (int l = 2; l <= RLOG; ++l) {
    sg[l] = (tl >> (l - 2)) & 1 ? -1.0f : 1.0f;
    in[l] = (tl & ((1 << (l - 2)) - 1)) == 0;
    whole[l] = !RAG || 2 * (tl & ~((1 << (l - 1)) - 1)) + (1 << (l - 1)) < m;
  }
  // channel c of this lane: va its level-1 difference, vb its other row (not normalised; RAG: scaled at every level)
  auto transform = [&](const u4 (&w)[2][CPR], int c, float& va, float& vb) __attribute__((always_inline)) {
    float x[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if constexpr (BF16) x[t] = (c & 1) ? bf16hi(w[t][c >> 3][(c >> 1) & 3]) : bf16lo(w[t][c >> 3][(c >> 1) & 3]);
      else x[t] = __uint_as_float(w[t][BF16 ? 0 : c >> 2][c & 3]);
    }
    float s = __fadd_rn(x[0], x[1]);
    va = __fsub_rn(x[0], x[1]);
    if constexpr (RAG) {
      s = 2 * tl + 1 < m ? __fmul_rn(s, kInvSqrt2) : x[0];
      va = __fmul_rn(va, kInvSqrt2);
    }
    auto level = [&](auto l_tag) __attribute__((always_inline)) {
      constexpr int l = decltype(l_tag)::value;
      if constexpr (l <= RLOG) {
        // lower lane: own + partner's, upper lane: partner's - own (the product is exact)
        float r = __builtin_fmaf(s, sg[l], partner<l>(s));
        if constexpr (RAG) {
          r = __fmul_rn(r, kInvSqrt2);
          s = in[l] && (whole[l] || sg[l] < 0.0f) ? r : s;
        } else {
          s = l == 2 || in[l] ? r : s;
        }
      }
    };
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});
    level(std::integral_constant<int, 4>{});
    vb = s;
  };
  float ra[32], rb[NG][32];  // rows A and B
  uint32_t pos[2] = {0u, 0u}, neg[2] = {0u, 0u};
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    RowMax<ASYM> ma, mb;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      if ((c & 7) == 0) __builtin_amdgcn_sched_barrier(0);  // the loaded words give way to the rows
      float va, vb;
      transform(raw[g], c, va, vb);
      ra[c] = va;
      rb[g][c] = vb;
      ma.template add<false>(c, va);
      mb.template add<NANMAX>(c, vb);
    }
    if constexpr (NG == 2) {
      if (g == 0) {  // (they do not fit the registers beside the second group's)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          *reinterpret_cast<float4*>(s_row + (i * (int)blockDim.x + tid) * 16) = make_float4(ra[4 * i], ra[4 * i + 1], ra[4 * i + 2], ra[4 * i + 3]);
      }
    }
    // lanes beyond d_in: the asymmetric form's keys must not see them (in the symmetric one their duplicates change nothing)
    const bool live = !ASYM || c0[g] < a.d;
    pos[0] = max(pos[0], live ? ma.pos() : 0u);
    pos[1] = max(pos[1], live ? mb.pos() : 0u);
    if constexpr (ASYM) {
      neg[0] = max(neg[0], live ? ma.neg() : 0u);
      neg[1] = max(neg[1], live ? mb.neg() : 0u);
    }
    if constexpr (NANMAX) {
      if (mb.nan != 0.0f && tl == 0 && live) {  // rare
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          pos[1] = max(pos[1], ASYM ? fkey(rb[g][i]) : absbits(rb[g][i]));
          if constexpr (ASYM) neg[1] = max(neg[1], fkey(-rb[g][i]));
        }
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    pos[h] = across_groups<NL>(pos[h]);
    if constexpr (ASYM) neg[h] = across_groups<NL>(neg[h]);
    if (lane < NL) {
      s_max[0][h * NL + tl][wave] = pos[h];
      if constexpr (ASYM) s_max[1][h * NL + tl][wave] = neg[h];
    }
  }
  __syncthreads();
  auto reduce = [&](int sign, int row) { return max_of_waves(s_max[sign][row], nw); };
  // the two rows of this lane: level (0: no norm), position in the plan's block, row of the sequence (RAG: STaMP slot, < 0: no
  // such coefficient)
  const int z2 = tl == 0 ? RLOG : __builtin_ctz((unsigned)tl) + 2;  // level of row B (the block sum: that of the last difference)
  const int R = RAG ? RK : a.R;
  const int ea = (R >> 1) + NL * part + tl, eb = tl == 0 ? 0 : (R >> z2) + (RK >> z2) * part + (tl >> (z2 - 1));
  const int sa = RAG ? (left_out ? -1 : stamp_rag_slot(a.rag, j, ea)) : j * R + ea;
  const int sb = RAG ? (left_out ? (tl == 0 ? 0 : -1) : stamp_rag_slot(a.rag, j, eb)) : j * R + eb;
  const int top_slot = RAG ? (left_out ? 0 : a.rag.o + j) : j;
  const bool sum_out = !RAG && a.abot != nullptr, row8 = !sum_out && top_slot < a.khi;  // (uniform)
  const float na = RAG ? 1.0f : kInvSqrt2, nb = RAG ? 1.0f : haar_norm(z2);
  const float qb = ASYM ? (tl == 0 && row8 ? 255.0f : 15.0f) : (tl == 0 && row8 ? 127.0f : 7.0f);
  float scale_a, inv_a, za, scale_b, inv_b, zb;
  if constexpr (ASYM) {
    row_params<true>(__fmul_rn(fkey_inv(reduce(0, tl)), na), __fmul_rn(fkey_inv(reduce(1, tl)), na), 15.0f, scale_a, inv_a, za);
    row_params<true>(__fmul_rn(fkey_inv(reduce(0, NL + tl)), nb), __fmul_rn(fkey_inv(reduce(1, NL + tl)), nb), qb, scale_b, inv_b, zb);
  } else {
    row_params<false>(__fmul_rn(__uint_as_float(reduce(0, tl)), na), 0.0f, 7.0f, scale_a, inv_a, za);
    row_params<false>(__fmul_rn(__uint_as_float(reduce(0, NL + tl)), nb), 0.0f, qb, scale_b, inv_b, zb);
  }
  if (tid < NL) {
    if (sa >= 0) {
      a.scales[seq0 + sa] = scale_a;
      if constexpr (ASYM) a.scales[a.zeros_off + seq0 + sa] = za;
    }
    if (sb >= 0 && !(sum_out && tl == 0)) {
      a.scales[seq0 + sb] = scale_b;
      if constexpr (ASYM) a.scales[a.zeros_off + seq0 + sb] = zb;
    }
  }
  // differences of even levels: their norm, a power of two, is part of the multiplier
  const bool fold = !RAG && tl != 0 && (z2 & 1) == 0;
  const float mb_ = fold ? __fmul_rn(inv_b, nb) : inv_b, nb_ = fold ? 1.0f : nb;
  const size_t brow = RAG ? ((size_t)b * a.rag.nb + j) * RK : seq0 + (size_t)j * R;
  uint8_t* const out = a.a6 + (brow >> 8) * (size_t)a.KT * kStageA6;
  const uint32_t row_a = (uint32_t)(brow & 255) + (uint32_t)ea, row_b = (uint32_t)(brow & 255) + (uint32_t)eb;
  uint32_t off_a, off_b;
  bool half_a, half_b;
  auto places = [&](int gb) __attribute__((always_inline)) {
    off_a = row_off6(row_a, gb);
    off_b = row_off6(row_b, gb);
    half_a = row_half6(row_a, gb);
    half_b = row_half6(row_b, gb);
  };
  if (RAG || parts == 1) places(RLOG);  // (most of it then depends on the block alone)
  else places(a.gb);
  auto place = [&](uint32_t off, int c) { return out + (chan_off6((uint32_t)c, kStageA6) + off); };
  // codes of 16 values; shift: what the stored code is below the unsigned one
  auto code = [&](const float (&x)[32], int odd, float n, float mul, float z, bool two) __attribute__((always_inline)) {
    f16v v;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = __fmul_rn(two ? __fmul_rn(x[2 * i + odd], n) : x[2 * i + odd], mul);
      v[i] = ASYM ? __builtin_amdgcn_fmed3f(__fadd_rn(rintf(p), z - 8.0f), -8.0f, 7.0f) : p;
    }
    return v;
  };
#pragma unroll
  for (int g = NG - 1; g >= 0; --g) {
    const int c = c0[g];
    const bool active = c < a.d;
    if constexpr (NG == 2) {
      if (g == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float4 v = *reinterpret_cast<const float4*>(s_row + (i * (int)blockDim.x + tid) * 16);
          ra[4 * i] = v.x;
          ra[4 * i + 1] = v.y;
          ra[4 * i + 2] = v.z;
          ra[4 * i + 3] = v.w;
        }
      }
    }
    const u6v wa = to_e2m3(code(ra, 0, na, inv_a, za, !RAG), code(ra, 1, na, inv_a, za, !RAG));
    if (active && (!RAG || sa >= 0)) store24(place(off_a, c), wa, half_a);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int c = c0[g];
    const bool active = c < a.d;
    if (sum_out) {
      if (active && tl == 0) {
        float4* o = reinterpret_cast<float4*>(a.abot + ((size_t)b * (a.s >> RLOG) + unit) * a.d + c);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = make_float4(rb[g][4 * i], rb[g][4 * i + 1], rb[g][4 * i + 2], rb[g][4 * i + 3]);
      }
    } else if (row8) {
      if (active && tl == 0) {
        const float qlo = ASYM ? 0.0f : -127.0f, qhi = ASYM ? 255.0f : 127.0f, shift = ASYM ? 128.0f : 0.0f;
        f16v qe, qo;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float te = RAG ? rb[g][2 * i] : __fmul_rn(rb[g][2 * i], nb), to = RAG ? rb[g][2 * i + 1] : __fmul_rn(rb[g][2 * i + 1], nb);
          qe[i] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(te, inv_b)), zb), qlo), qhi) - shift;
          qo[i] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(to, inv_b)), zb), qlo), qhi) - shift;
        }
        store_hi24(a.hi6, b * a.khi + top_slot, a.KT, qe, qo, c);
      }
    }
    const u6v wb = to_e2m3(code(rb[g], 0, nb_, mb_, zb, !RAG), code(rb[g], 1, nb_, mb_, zb, !RAG));
    if (active && (!RAG || sb >= 0) && !(tl == 0 && (sum_out || row8))) store24(place(off_b, c), wb, half_b);
  }
}

// up to ML levels of the in-place network
template <int NN, int ML>
__device__ __forceinline__ void top_network(float (&v)[NN], int lv) {
#pragma unroll
  for (int l = 1; l <= ML; ++l)
    if (l <= lv) {
#pragma unroll
      for (int i = 0; i < NN; i += 1 << l) {
        const float x = v[i], y = v[i + (1 << (l - 1))];
        v[i] = __fadd_rn(x, y);
        v[i + (1 << (l - 1))] = __fsub_rn(x, y);
      }
    }
}
// its finished coefficients, normalised, to their STaMP slots; v[0] is sum q0 of `len`, LEV0 levels lie below.  last: what is
// left are the approximations.
template <int NN, int LEV0>
__device__ __forceinline__ void top_store(const float (&v)[NN], float* base, int d, int len, int q0, int lv, bool last) {
#pragma unroll
  for (int i = 0; i < NN; ++i) {
    const int l = i == 0 ? 32 : __builtin_ctz((unsigned)i) + 1;
    if (i < len) {
      if (l <= lv) base[(size_t)((len >> l) + ((q0 + i) >> l)) * d] = __fmul_rn(v[i], haar_norm(LEV0 + l));
      else if (last) base[(size_t)((q0 + i) >> lv) * d] = __fmul_rn(v[i], haar_norm(LEV0 + lv));
    }
  }
}
// The levels above parts of 8 tokens, in place over their n sums (16 to 512) of every channel.  A thread holds 16 neighbouring
// sums of one channel and runs up to four levels on them; what is left of each group meets in LDS, where one thread per channel runs
// the rest.  2048 tokens x 4096 channels (256 sums): 17.3 us with every level and the rows' maxima in LDS (k_top).
template <int CH>
__global__ __launch_bounds__(1024) void k_top_parts(float* __restrict__ abot, int n, int d, int levels) {
  __shared__ float s_sum[32][CH];
  const int tid = threadIdx.x, ch = tid % CH, g = tid / CH, c = (int)blockIdx.x * CH + ch, ng = n >> 4;
  const bool active = c < d;
  float* const base = abot + (size_t)blockIdx.y * n * d + min(c, d - 1);
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = base[(size_t)(16 * g + i) * d];
  const int lv = min(levels, 4), rest = levels - lv;
  top_network<16, 4>(v, lv);
  s_sum[g][ch] = v[0];
  __syncthreads();  // (and every row has been read before the first is overwritten)
  if (active) top_store<16, 3>(v, base, d, n, 16 * g, lv, rest == 0);
  if (rest == 0 || g != 0 || !active) return;
  float w[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) w[i] = i < ng ? s_sum[i][ch] : 0.0f;
  top_network<32, 5>(w, rest);
  top_store<32, 7>(w, base, d, ng, 0, rest, true);
}

// One row of those levels, a lane 32 channels: slots below k are 8-bit rows, the others differences of the plan's blocks.
template <bool ASYM>
__global__ __launch_bounds__(256) void k_quant_parts(const float* __restrict__ T, const LaneArgs a) {
  __shared__ uint32_t s_red[8];
  const int slot = blockIdx.x, b = blockIdx.y, n = a.s >> 3, tid = threadIdx.x, nw = (int)(blockDim.x >> 6);
  const int c = tid * 32, cl = min(c, a.d - 32);
  const size_t trow = (size_t)b * n + slot;
  float x[32];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float4 v = *reinterpret_cast<const float4*>(T + trow * a.d + cl + 4 * i);
    x[4 * i] = v.x;
    x[4 * i + 1] = v.y;
    x[4 * i + 2] = v.z;
    x[4 * i + 3] = v.w;
  }
  const bool row8 = slot < a.k, active = c < a.d;
  // (maxima as where these rows came from before: a NaN is the largest of a top row)
  uint32_t mp = 0u, mn = 0u;
  if (row8) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      mp = max(mp, ASYM ? fkey(x[i]) : absbits(x[i]));
      if constexpr (ASYM) mn = max(mn, fkey(-x[i]));
    }
  } else {
    RowMax<ASYM> m;
#pragma unroll
    for (int i = 0; i < 32; ++i) m.template add<false>(i, x[i]);
    mp = m.pos();
    if constexpr (ASYM) mn = m.neg();
  }
  mp = wave_max_u32(active ? mp : 0u);
  mn = wave_max_u32(active ? mn : 0u);
  if ((tid & 63) == 0) {
    s_red[tid >> 6] = mp;
    s_red[4 + (tid >> 6)] = mn;
  }
  __syncthreads();
  for (int i = 0; i < nw; ++i) {
    mp = max(mp, s_red[i]);
    mn = max(mn, s_red[4 + i]);
  }
  const float qmax = ASYM ? (row8 ? 255.0f : 15.0f) : (row8 ? 127.0f : 7.0f);
  float scale, inv, z;
  if constexpr (ASYM) row_params<true>(fkey_inv(mp), fkey_inv(mn), qmax, scale, inv, z);
  else row_params<false>(__uint_as_float(mp), 0.0f, qmax, scale, inv, z);
  // slot k 2^m + i: block i >> m, position 2^m + i % 2^m
  const int m = row8 ? 0 : 31 - __builtin_clz((unsigned)(slot / a.k)), i = row8 ? 0 : slot - (a.k << m);
  const int row = row8 ? slot * a.R : (i >> m) * a.R + (1 << m) + (i & ((1 << m) - 1));
  const size_t srow = (size_t)b * a.s + row;
  if (tid == 0) {
    a.scales[srow] = scale;
    if constexpr (ASYM) a.scales[a.zeros_off + srow] = z;
  }
  f16v ev, od;
  const float qlo = ASYM ? 0.0f : -qmax, shift = ASYM ? (row8 ? 128.0f : 8.0f) : 0.0f;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    ev[q] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(x[2 * q], inv)), z), qlo), qmax) - shift;
    od[q] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(x[2 * q + 1], inv)), z), qlo), qmax) - shift;
  }
  if (!active) return;
  if (row8) {
    store_hi24(a.hi6, b * a.k + slot, a.KT, ev, od, c);
  } else {
    const uint32_t mr = (uint32_t)(srow & 255);
    store24(a.a6 + (srow >> 8) * (size_t)a.KT * kStageA6 + (chan_off6((uint32_t)c, kStageA6) + row_off6(mr, a.gb)), to_e2m3(ev, od),
            row_half6(mr, a.gb));
  }
}

// Rows as they are (plans without transform, transformed tokens of the general path): a lane holds 32 channels of one row, a
// workgroup ROWS rows (unit_of_block: 64 neighbouring ones share an XCD, whose L2 gathers their lines of the operand).  The first k rows of a sequence are
// 8-bit rows.  Each value is read once.  What bounds it: the launch and its first loads on few rows, memory on many.
// 2048 rows x 4096 channels fp32 8.6 us (a workgroup per row that reads it twice and stores 8 bytes at a time: 14.2),
// 262144 x 256 bf16, the whole layer with 256 outputs, 75 (packed codes and a pass that converts them 188).
template <int ROWS, bool BF16, bool ASYM>
__global__ __launch_bounds__(1024) void k_lanes_rows(const LaneArgs a, int rows) {
  constexpr int CPR = BF16 ? 4 : 8;
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][ROWS][16];  // [sign][row][wave]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
  const int tl = lane & (ROWS - 1), m = unit_of_block<ROWS>(blockIdx.x, gridDim.x) * ROWS + tl, mr = min(m, rows - 1);
  const int c = (wave * (64 / ROWS) + lane / ROWS) * 32, cl = min(c, a.d - 32);
  u4 raw[CPR];
  const uint8_t* const src = reinterpret_cast<const uint8_t*>(a.X) + ((size_t)mr * a.d + cl) * (BF16 ? 2 : 4);
#pragma unroll
  for (int h = 0; h < CPR; ++h) raw[h] = *reinterpret_cast<const u4*>(src + 16 * h);
  float x[32];
  RowMax<ASYM> mx;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if constexpr (BF16) x[i] = (i & 1) ? bf16hi(raw[i >> 3][(i >> 1) & 3]) : bf16lo(raw[i >> 3][(i >> 1) & 3]);
    else x[i] = __uint_as_float(raw[BF16 ? 0 : i >> 2][i & 3]);
    mx.template add<false>(i, x[i]);
  }
  const bool live = !ASYM || c < a.d;
  const uint32_t pos = across_groups<ROWS>(live ? mx.pos() : 0u);
  uint32_t neg = 0u;
  if constexpr (ASYM) neg = across_groups<ROWS>(live ? mx.neg() : 0u);
  if (lane < ROWS) {
    s_max[0][tl][wave] = pos;
    if constexpr (ASYM) s_max[1][tl][wave] = neg;
  }
  __syncthreads();
  auto reduce = [&](int sign) { return max_of_waves(s_max[sign][tl], nw); };
  const int b = mr / a.s, pr = mr - b * a.s;
  const bool row8 = pr < a.k;
  const float qmax = ASYM ? (row8 ? 255.0f : 15.0f) : (row8 ? 127.0f : 7.0f);
  float scale, inv, z;
  if constexpr (ASYM) row_params<true>(fkey_inv(reduce(0)), fkey_inv(reduce(1)), qmax, scale, inv, z);
  else row_params<false>(__uint_as_float(reduce(0)), 0.0f, qmax, scale, inv, z);
  if (tid < ROWS && m < rows) {
    a.scales[m] = scale;
    if constexpr (ASYM) a.scales[a.zeros_off + m] = z;
  }
  const float qlo = ASYM ? 0.0f : -qmax, shift = ASYM ? (row8 ? 128.0f : 8.0f) : 0.0f;
  f16v ev, od;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float p = __fmul_rn(x[2 * i], inv), q = __fmul_rn(x[2 * i + 1], inv);
    ev[i] = __builtin_amdgcn_fmed3f(__fadd_rn(rintf(p), z), qlo, qmax) - shift;
    od[i] = __builtin_amdgcn_fmed3f(__fadd_rn(rintf(q), z), qlo, qmax) - shift;
  }
  if (c >= a.d || m >= rows) return;
  if (row8) {
    store_hi24(a.hi6, b * a.k + pr, a.KT, ev, od, c);
  } else {
    store24(a.a6 + (size_t)(m >> 8) * a.KT * kStageA6 + (chan_off6((uint32_t)c, kStageA6) + row_off6((uint32_t)m & 255, 2)), to_e2m3(ev, od),
            row_half6((uint32_t)m, 2));
  }
}

template <int ROWS, bool BF16>
void launch_rows(bool asym, const LaneArgs& a, int rows, hipStream_t st) {
  const dim3 grid((rows + ROWS - 1) / ROWS), blk((a.d * ROWS + 2047) / 2048 * 64);
  if (asym) hipLaunchKernelGGL((k_lanes_rows<ROWS, BF16, true>), grid, blk, 0, st, a, rows);
  else hipLaunchKernelGGL((k_lanes_rows<ROWS, BF16, false>), grid, blk, 0, st, a, rows);
}

template <int RLOG, bool BF16, bool ASYM, bool RAG>
hipError_t launch_n(const LaneArgs& a, int blocks, int B, hipStream_t st) {
  constexpr int CW = 64 / (1 << (RLOG - 1)) * 32;  // channels of a wave
  const int waves = (a.d + CW - 1) / CW;
  const dim3 grid(blocks, B);
  const bool nan_max = !RAG && a.d > (BF16 ? 8192 : 4096);  // as the streaming kernels with split channels
  if (waves > 16) {
    if constexpr (BF16 && !RAG && RLOG == 3) {
      if (waves > 24 || !nan_max) return hipErrorInvalidValue;
      const int threads = (waves + 1) / 2 * 64;
      const size_t lds = (size_t)threads * 128;
      static size_t lds_done[kStampMaxDevices] = {};
      const hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_lanes1d<RLOG, BF16, ASYM, false, 2, true>), lds, lds_done);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((k_lanes1d<RLOG, BF16, ASYM, false, 2, true>), grid, dim3(threads), lds, st, a);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if constexpr (!RAG && RLOG == 3) {
    if (nan_max) {
      hipLaunchKernelGGL((k_lanes1d<RLOG, BF16, ASYM, false, 1, true>), grid, dim3(waves * 64), 0, st, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_lanes1d<RLOG, BF16, ASYM, RAG, 1, false>), grid, dim3(waves * 64), 0, st, a);
  return hipGetLastError();
}
template <int RLOG, bool RAG>
hipError_t launch(const LaneArgs& a, int x_bf16, int asym, int blocks, int B, hipStream_t st) {
  if (x_bf16) return asym ? launch_n<RLOG, true, true, RAG>(a, blocks, B, st) : launch_n<RLOG, true, false, RAG>(a, blocks, B, st);
  return asym ? launch_n<RLOG, false, true, RAG>(a, blocks, B, st) : launch_n<RLOG, false, false, RAG>(a, blocks, B, st);
}

}  // namespace

// Plans that these kernels serve: the channels fit one workgroup; more than its 16 waves hold in one group of 32 per lane only
// where the blocks fill more than half of the CUs (2 against 1 pass over X: 512 x 11008 16.1 us in two passes over split channels,
// 17.7 here, 1024: 17.1, 17.8, 2048: 32.5, 21.5, 4096 (min-max codes): 66.6, 35.8).
bool stamp_lanes1d_fits(const stamp_plan* p, int rlog) {
  const StampGeom& g = p->geom;
  if (g.d < 64) return false;  // two of a wave's 64 lanes per token pair: 16 x 1024 tokens x 32 18.8 us streaming, 19.2 here
  if (rlog == 4) return g.d <= 4096;
  if (rlog != 3) return false;
  if (g.d <= 8192) return true;
  return g.x_bf16 && !p->rag.on && g.d <= 12288 && (int64_t)g.B * g.s > 4 * stamp_device_cus();
}

hipError_t stamp_launch_lanes1d(const stamp_plan* p, int rlog, const void* X, uint8_t* a6, float* scales, float* abot, const StampHiOut& hi,
                                hipStream_t st) {
  const StampGeom& g = p->geom;
  LaneArgs a = {};
  a.X = X;
  a.a6 = a6;
  a.scales = scales;
  a.abot = abot;
  a.R = g.R;
  a.s = g.s;
  a.d = g.d;
  a.k = g.k;
  a.khi = g.khi;
  a.KT = p->Kpad >> 7;
  a.zeros_off = (size_t)g.B * g.s;
  a.hi6 = hi;
  a.rag = p->rag;
  a.gb = stamp_row_group_bit(p);
  if (p->rag.on) {
    const int blocks = p->rag.nb + p->rag.o;
    return rlog == 3 ? launch<3, true>(a, g.x_bf16, g.asym, blocks, g.B, st) : launch<4, true>(a, g.x_bf16, g.asym, blocks, g.B, st);
  }
  return rlog == 3 ? launch<3, false>(a, g.x_bf16, g.asym, g.s / 8, g.B, st) : launch<4, false>(a, g.x_bf16, g.asym, g.s / 16, g.B, st);
}

hipError_t stamp_launch_top_parts(const stamp_plan* p, float* abot, uint8_t* a6, float* scales, const StampHiOut& hi, hipStream_t st) {
  const StampGeom& g = p->geom;
  const int n = g.s / 8, ng = n / 16, levels = g.L + g.r - 3, threads = (g.d / 32 + 63) / 64 * 64;
  if (n < 16 || n > 512 || threads > 256) return hipErrorInvalidValue;
  // 32 channels per workgroup (whole lines of a row) where that fills the CUs, else 16
  if (g.d / 32 * g.B >= stamp_device_cus()) hipLaunchKernelGGL(k_top_parts<32>, dim3((g.d + 31) / 32, g.B), dim3(32 * ng), 0, st, abot, n, g.d, levels);
  else hipLaunchKernelGGL(k_top_parts<16>, dim3((g.d + 15) / 16, g.B), dim3(16 * ng), 0, st, abot, n, g.d, levels);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LaneArgs a = {};
  a.a6 = a6;
  a.scales = scales;
  a.s = g.s;
  a.d = g.d;
  a.k = g.k;
  a.KT = p->Kpad >> 7;
  a.R = g.R;
  a.gb = stamp_row_group_bit(p);
  a.zeros_off = (size_t)g.B * g.s;
  a.hi6 = hi;
  if (g.asym) hipLaunchKernelGGL(k_quant_parts<true>, dim3(n, g.B), dim3(threads), 0, st, abot, a);
  else hipLaunchKernelGGL(k_quant_parts<false>, dim3(n, g.B), dim3(threads), 0, st, abot, a);
  return hipGetLastError();
}

hipError_t stamp_launch_lanes_rows(const stamp_plan* p, const void* X, int x_bf16, uint8_t* a6, float* scales, const StampHiOut& hi, hipStream_t st) {
  const StampGeom& g = p->geom;
  LaneArgs a = {};
  a.X = X;
  a.a6 = a6;
  a.scales = scales;
  a.s = g.s;
  a.d = g.d;
  a.k = g.k;
  a.KT = p->Kpad >> 7;
  a.zeros_off = (size_t)g.B * g.s;
  a.hi6 = hi;
  const int rows = g.B * g.s;
  // as many rows as 1024 threads hold, two where four leave CUs without a workgroup (WHT of 256 x 1312, layer to 512: 34.4 with four, 33.5;
  // 1024 x 4096 55.4, 55.5, 2048 x 4096 66.0, 67.0)
  const int n = g.d <= 8192 && rows > 2 * stamp_device_cus() ? 4 : (g.d <= 16384 ? 2 : 1);
  if (n == 4) x_bf16 ? launch_rows<4, true>(g.asym, a, rows, st) : launch_rows<4, false>(g.asym, a, rows, st);
  else if (n == 2) x_bf16 ? launch_rows<2, true>(g.asym, a, rows, st) : launch_rows<2, false>(g.asym, a, rows, st);
  else x_bf16 ? launch_rows<1, true>(g.asym, a, rows, st) : launch_rows<1, false>(g.asym, a, rows, st);
  return hipGetLastError();
}
