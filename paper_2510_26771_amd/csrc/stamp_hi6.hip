// The 8-bit rows of the STaMP linear layer when the whole batch has few of them: their GEMM on the FP6 matrix pipeline
// (operands as in stamp_hi6.h), dequantization, the top levels of the inverse transform, and the store of the block sums P
// (or of the rows themselves), one kernel.
//
// The GEMM is a stream of the weights (0.75 byte each) against a few rows that come from L2: bound by how many bytes are
// in flight, so nothing is staged.  Every wave reads its operands straight from memory into registers (the layout makes a
// wave's 16-byte loads 1 KB of consecutive addresses), the eight waves of a workgroup split the depth (two groups of four
// when there are more than 64 rows: each group takes 64), and only their sums meet in LDS.  The sums are whole numbers and
// stay whole: fp32 holds each FP6 sum exactly, 16 h + l and the sum over the waves are int32.
// Measured (rows x depth x d_out, microseconds; before: int8 GEMM + top levels of the inverse as a kernel of its own):
// 64 x 4096 x 11008: 15.3 (16.1 + 10.1), 128 x 4096 x 4096: 11.9 (17.8 + 11.9), 64 x 11008 x 4096: 16.9 (19.1 + 4.8),
// 128 x 1152 x 4608: 8.2 (15.7 + 5.2), 512 x 4096 x 4096: 33 (34 + 15).
#include "stamp_hi6.h"

namespace {

using namespace stamp_gemm;

// register = integer sum / 64 after the sums have met
struct AccHi6 {
  static constexpr bool kLoRows = false;
  static constexpr float kZeroShift = 128.0f;
  static constexpr float kToAcc = 1.0f;
};

struct Hi6Args {
  GemmArgs a;        // A: packed rows, Bq: FP6 weights, M rows, g.k rows per sequence, scales, sw, colsum, bias, rag
  int np, ng;        // 32-row pairs per wave, row groups per workgroup
  int mode;          // 0: block sums -> out [M][ld_out] (g.L top levels inverted), 1: rows -> Y + bias (plans without transform),
                     // 2: rows -> fp32 rows b * g.s + slot of out, 3: blocked form of any length (StampRag): as 0 times norm, slot < o -> Y
  float norm;        // mode 3
  void* Y;           // mode 3
  const float *sa, *sw;  // GRP: [row group][K step][rows][2], [column tile][K step][4 blocks][32][2]
};

// place of a sum in its wave's part (NC = 2: col = the column, else its place in the strip): the four lane groups of a wave write
// rows 8 apart, to 16 banks each
template <int NC>
__device__ __forceinline__ int part_at(int row, int col) {
  const int b3 = (row >> 3) & 1, b4 = (row >> 4) & 1;
  return NC == 2 ? row * 64 + (col ^ b3 ^ (b4 << 5)) : (row ^ b4) * 32 + (col ^ (b3 << 4));
}

// GRP: one scale per 64 channels (a half of a K step) and row / column: the sums are rescaled half by half, s_part holds fp32
// AHEAD: the next step's operands are in flight while a step is multiplied.  That takes twice the registers, so it is for
// launches that leave no CU a second workgroup: 64 x 11008 x 4096 (128 workgroups) 16.9 us against 18.9, 128 x 4096 x 4096
// (256) 11.9 against 12.8, but 64 x 4096 x 11008 (344) 21.4 against 17.4.  Up to 32 rows: WHT layer of 512 x 4096 -> 1024 43.0
// without, 41.0 with, 2048 x 4096 -> 4096 81.3, 78.8.
// NC: strips of 32 columns per workgroup.  Two: the rows' operand, the larger share of what a CU's vector memory path moves (64 bytes a
// clock: that path is what bounds the loop), is read half as often, but nothing covers a workgroup's start and end (the rule:
// stamp_hi6_two_strips).  64 x 4096 x 11008 16.2 us with one, 15.3 with two, of which the loop 8, the launch and the sums of the waves 5, the top levels 2.
template <int NP, bool GRP, bool AHEAD, int NC = 1>
__global__ __launch_bounds__(512, AHEAD || NC == 2 ? 2 : 4) void k_hi6(const Hi6Args h) {
  const GemmArgs& a = h.a;
  const StampGeom& g = a.g;
  constexpr int C = 32 * NC, RW = 32 * NP, RS = 512 / C;  // columns, rows of a wave; rows apart that a thread finishes
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  int* const s_part = reinterpret_cast<int*>(smem);            // [8 waves][RW][C]
  __shared__ __attribute__((aligned(16))) uint8_t s_info[kRowInfoBytes];
  __shared__ int s_pos[128];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kg = lane >> 5;
  const int KT = a.Kpad / BK, kw = 8 / h.ng, rg = wave / kw, kp = wave - rg * kw;
  const int RG = RW * h.ng, m0 = (int)blockIdx.y * RG;  // rows of the workgroup
  // strip of 32 columns: block `st` of the weight layout = columns 64 (st / 2) + 2 l + st % 2
  const int st = NC * (int)blockIdx.x;
  const uint8_t* pb = a.Bq + (size_t)(st >> 2) * KT * kStageB6 + (st & 3) * kBlock6;
  const uint8_t* pa = a.A + (size_t)((int)blockIdx.y * h.ng + rg) * KT * (2 * NP * kBlock6);
  const uint32_t lane16 = (uint32_t)lane * 16u;
  const int kt0 = KT * kp / kw, kt1 = KT * (kp + 1) / kw;

  // GRP: MFMA blocks of 32 x 32; else four tiles of 16 x 16 per block, 2 tc + th as in the 4-bit rows' GEMM
  v16f acc[GRP ? NP : 1];
  f4 acct[NC][GRP ? 1 : 2 * NP][4];
  if constexpr (GRP) {
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
  } else {
#pragma unroll
    for (int s = 0; s < NC; ++s)
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) acct[s][i][q] = (f4){0.0f, 0.0f, 0.0f, 0.0f};
  }
  [[maybe_unused]] auto multiply1 = [&](f4 (&c)[4], const Frag6& b, const Frag6& f) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      c[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4((q & 1) ? f.h1() : f.h0(), (q & 2) ? b.h1() : b.h0(), c[q], 2, 2, 0, 0, 0, 0);
  };
  [[maybe_unused]] auto multiply = [&](const Frag6& b, const Frag6 (&f)[2 * NP]) __attribute__((always_inline)) {
    if constexpr (!GRP) {
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i) multiply1(acct[0][i], b, f[i]);
    }
  };
  if (!GRP && tid < RG) {
    float fac = 0.0f, rz = 0.0f;
    int dst = -1;
    compute_row_info<AccHi6, 1>(a, m0, tid, fac, dst, rz);
    write_row_info(s_info, tid, fac, dst, rz);
  }
  if constexpr (NC == 2) {
    for (int kt = kt0; kt < kt1; ++kt) {
      Frag6 fb[NC], fa[2 * NP];
#pragma unroll
      for (int s = 0; s < NC; ++s) fb[s].load(pb + (size_t)kt * kStageB6 + s * kBlock6, lane16);
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i) fa[i].load(pa + (size_t)kt * (2 * NP * kBlock6) + i * kBlock6, lane16);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i)
#pragma unroll
        for (int s = 0; s < NC; ++s) multiply1(acct[s][i], fb[s], fa[i]);
    }
  }
  // Neither: at most 128 registers, four waves per SIMD (two workgroups per CU) hide each other's loads.
  if constexpr (AHEAD) {
    Frag6 fb[2], fa[2][2 * NP];
    auto fetch = [&](int kt, Frag6& b, Frag6 (&f)[2 * NP]) {
      b.load(pb + (size_t)kt * kStageB6, lane16);
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i) f[i].load(pa + (size_t)kt * (2 * NP * kBlock6) + i * kBlock6, lane16);
    };
    int kt = kt0;
    if (kt < kt1) {
      fetch(kt, fb[0], fa[0]);
      for (; kt + 2 < kt1; kt += 2) {
        fetch(kt + 1, fb[1], fa[1]);
        __builtin_amdgcn_sched_barrier(0);  // (its loads would be put off one by one)
        multiply(fb[0], fa[0]);
        __builtin_amdgcn_sched_barrier(0);
        fetch(kt + 2, fb[0], fa[0]);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fb[1], fa[1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (kt + 1 < kt1) fetch(kt + 1, fb[1], fa[1]);
      __builtin_amdgcn_sched_barrier(0);
      multiply(fb[0], fa[0]);
      if (kt + 1 < kt1) multiply(fb[1], fa[1]);
    }
  }
  for (int kt = AHEAD || NC == 2 ? kt1 : kt0; kt < kt1; ++kt) {
    Frag6 fb, fa[2 * NP];
    const uint8_t* const ra = pa + (size_t)kt * (2 * NP * kBlock6);
    fb.load(pb + (size_t)kt * kStageB6, lane16);
    constexpr int first = GRP ? 2 * NP : 2;
#pragma unroll
    for (int i = 0; i < first; ++i) fa[i].load(ra + i * kBlock6, lane16);
    if constexpr (GRP) {
      // S = row scale times column scale (k = 1 of the product is zero)
      const f2 sw = reinterpret_cast<const f2*>(h.sw)[((size_t)(st >> 2) * KT + kt) * 128 + (st & 3) * 32 + l32];
      const v16f zero = {};
#pragma unroll
      for (int pr = 0; pr < NP; ++pr) {
        const f2 sa = reinterpret_cast<const f2*>(h.sa)[((size_t)((int)blockIdx.y * h.ng + rg) * KT + kt) * RW + pr * 32 + l32];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const v16f th = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(hf ? fa[2 * pr].h1() : fa[2 * pr].h0(), hf ? fb.h1() : fb.h0(), zero, 2,
                                                                          2, 0, 0, 0, 0);
          const v16f tl = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(hf ? fa[2 * pr + 1].h1() : fa[2 * pr + 1].h0(),
                                                                          hf ? fb.h1() : fb.h0(), zero, 2, 2, 0, 0, 0, 0);
          const v16f S = __builtin_amdgcn_mfma_f32_32x32x2f32(kg == 0 ? sa[hf] : 0.0f, kg == 0 ? sw[hf] : 0.0f, zero, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[pr][v] = __builtin_fmaf(__builtin_fmaf(16.0f, th[v], tl[v]), S[v], acc[pr][v]);
        }
      }
    } else {
      // (the compiler would put the loads off to save registers and have four of them in flight: 3200 workgroups at depth 8192 189 us in place of 168,
      // 528 at depth 4096 25.1, 21.6; all fifteen do not fit)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i) {
        multiply1(acct[0][i], fb, fa[i]);
        if (i + first < 2 * NP) {
          __builtin_amdgcn_sched_barrier(0);
          fa[i + first].load(ra + (i + first) * kBlock6, lane16);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  // staging position of a row: its natural position among the block sums of its sequence (top levels), else the row itself
  if (h.mode == 0 && g.L > 0) {
    if (tid < RG) {
      const int seq = tid / g.k, q = tid - seq * g.k;
      int e, lvl;
      if (!g.is2d) e = stamp_top_slot_1d(q, g.k, g.L, &lvl);
      else e = stamp_top_slot_2d(q / g.G, q % g.G, g.G, g.L, &lvl);
      s_pos[seq * g.k + e] = tid;
    }
  }
#pragma unroll
  for (int pr = 0; pr < NP; ++pr)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if constexpr (GRP) {
        const int row = pr * 32 + 8 * (v >> 2) + 4 * kg + (v & 3);
        s_part[(wave * RW + row) * C + l32] = __float_as_int(acc[pr][v]);
      } else {
        const int q = v >> 2, row = pr * 32 + 8 * (lane >> 4) + 4 * (q & 1) + (v & 3), col = 16 * (q >> 1) + (lane & 15);
#pragma unroll
        for (int s = 0; s < NC; ++s)
          s_part[wave * RW * C + part_at<NC>(row, NC == 2 ? 2 * col + s : col)] =
              16 * (int)(acct[s][2 * pr][q][v & 3] * 64.0f) + (int)(acct[s][2 * pr + 1][q][v & 3] * 64.0f);
      }
    }
  __syncthreads();

  // sums over the waves, dequantized
  const float* s_fac = reinterpret_cast<const float*>(s_info);
  const float* s_rz = reinterpret_cast<const float*>(s_info + 2048);
  const int c = tid & (C - 1), r0 = tid / C;  // this thread: column c, rows r0, r0 + RS, ..
  const int n = NC == 2 ? 32 * st + c : 64 * (st >> 1) + 2 * c + (st & 1);
  const float swn = GRP ? 0.0f : a.sw[n], csn = !GRP && g.asym ? a.colsum[n] : 0.0f;
  float y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = r0 + RS * i;
    y[i] = 0.0f;
    if (r < RG) {
      const int base = (r / RW) * kw * RW * C + (GRP ? (r & (RW - 1)) * C + c : part_at<NC>(r & (RW - 1), c));
      if constexpr (GRP) {
        float sum = 0.0f;
        for (int q = 0; q < kw; ++q) sum += __int_as_float(s_part[base + q * (RW * C)]);
        if (m0 + r < a.M) y[i] = sum;
        continue;
      }
      int sum = 0;
      for (int q = 0; q < kw; ++q) sum += s_part[base + q * (RW * C)];
      const float af = g.asym ? __builtin_fmaf(-s_rz[r], csn, (float)sum) : (float)sum;
      if (m0 + r < a.M) y[i] = (af * s_fac[r]) * swn;
    }
  }
  if (h.mode == 0 && g.L > 0) {
    // top levels in LDS: same pairs in the same order as k_inverse_top
    float* const s_buf = reinterpret_cast<float*>(smem);  // [RG][C]
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (r0 + RS * i < RG) s_buf[s_pos[r0 + RS * i] * C + c] = y[i];
    __syncthreads();
    const int nseq = RG / g.k;
    if (!g.is2d) {
      for (int s2 = 1 << g.L; s2 >= 2; s2 >>= 1) {
        const int npair = RG / s2;
        for (int i = r0; i < npair; i += RS) {
          float *px = &s_buf[(i * s2) * C + c], *pd = &s_buf[(i * s2 + (s2 >> 1)) * C + c];
          const float x = *px, d = *pd;
          *px = x + d;
          *pd = x - d;
        }
        __syncthreads();
      }
    } else {
      for (int s2 = 1 << g.L; s2 >= 2; s2 >>= 1) {
        const int nc = g.G / s2, hf = s2 >> 1, cells = nc * nc;
        for (int i = r0; i < nseq * cells; i += RS) {
          const int seq = i / cells, q = i - seq * cells, cy = q / nc, cx = q - cy * nc;
          float* p00 = &s_buf[(seq * g.k + (cy * s2) * g.G + cx * s2) * C + c];
          float *p01 = p00 + hf * C, *p10 = p00 + hf * g.G * C, *p11 = p10 + hf * C;
          const float cLL = *p00, cW = *p01, cH = *p10, cD = *p11;
          const float t0 = cLL + cH, t2 = cLL - cH, t1 = cW + cD, t3 = cW - cD;
          *p00 = t0 + t1;
          *p01 = t0 - t1;
          *p10 = t2 + t3;
          *p11 = t2 - t3;
        }
        __syncthreads();
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (r0 + RS * i < RG) y[i] = s_buf[(r0 + RS * i) * C + c];
  }
  if (n >= a.N) return;
  float* const out = reinterpret_cast<float*>(a.out);
  const float bv = ((h.mode == 1 || h.mode == 3) && a.bias != nullptr) ? a.bias[n] : 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = r0 + RS * i, m = m0 + r;
    if (r >= RG || m >= a.M) continue;
    if (h.mode == 0) {
      out[(size_t)m * a.ld_out + n] = y[i];
    } else {
      const int b = m / g.k, slot = m - b * g.k;
      const size_t idx = ((size_t)b * g.s + slot) * a.N + n;
      if (h.mode == 2) {
        out[idx] = y[i];
      } else if (h.mode == 3 && slot >= a.rag.o) {
        out[(size_t)m * a.ld_out + n] = y[i] * h.norm;
      } else {
        const float v = y[i] + bv;
        void* Y = h.mode == 1 ? a.out : h.Y;
        if (g.y_bf16) reinterpret_cast<__bf16*>(Y)[idx] = (__bf16)v;
        else reinterpret_cast<float*>(Y)[idx] = v;
      }
    }
  }
}

template <int NP, bool GRP, bool AHEAD, int NC = 1>
hipError_t launch(const Hi6Args& h, hipStream_t st) {
  constexpr size_t lds = (size_t)8 * 32 * NP * 32 * NC * sizeof(int);
  static size_t lds_done[kStampMaxDevices] = {};
  const hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_hi6<NP, GRP, AHEAD, NC>), lds, lds_done);
  if (e != hipSuccess) return e;
  const int rows = 32 * NP * h.ng;
  hipLaunchKernelGGL((k_hi6<NP, GRP, AHEAD, NC>), dim3((h.a.N + 63) / 64 * (2 / NC), (h.a.M + rows - 1) / rows), dim3(512), lds, st, h);
  return hipGetLastError();
}

}  // namespace

// rows of this GEMM: all top rows of every sequence, or (own) the first khi of them
namespace {
int hi6_rows(const stamp_plan* p, int own) { return p->geom.B * (own ? p->geom.khi : p->geom.k); }
// 64 rows per workgroup (more workgroups, each with its waves' depth split eight ways), 128 where a sequence has that many
// top rows and its top levels are inverted here
int hi6_ng(const stamp_plan* p, int own) { return !p->geom.ident && !own && p->geom.L > 0 && p->geom.k > 64 ? 2 : 1; }
int hi6_strips(const stamp_plan* p) { return (p->geom.N + 63) / 64 * 2; }
// 32-row pairs of a wave: one for up to 32 rows, and where two would leave half of the CUs without a workgroup (unless a sequence's top
// levels need the rows together): more CUs then ask memory for the weights.  64 x 4096 x 4096 with weights that are not in the
// caches 14.0 us in 128 workgroups, 10.3 in 256; layers, WHT of 1024 x 2048 -> 2048 42.1, 39.3, 2 x 256 x 4096 -> 2048 45.4, 40.6; 4 x
// 300 tokens without transform, 1024 -> 768 21.9, 19.8.
int hi6_np(const stamp_plan* p, int own) {
  const int M = hi6_rows(p, own);
  if (M <= 32) return 1;
  const bool together = p->gen.group != 0 || (!p->geom.ident && !own && p->geom.L > 0 && p->geom.k > 32);
  return !together && 2 * hi6_strips(p) * ((M + 63) / 64) <= stamp_device_cus() ? 1 : 2;
}
}  // namespace

int stamp_hi6_rows_per_workgroup(const stamp_plan* p, int own) { return 32 * hi6_np(p, own) * hi6_ng(p, own); }
namespace {
int64_t hi6_groups(const stamp_plan* p, int own) {
  const int rows = stamp_hi6_rows_per_workgroup(p, own);
  return (hi6_rows(p, own) + rows - 1) / rows;
}
}  // namespace

// Two strips of columns a workgroup (n of them, one per CU) in place of one: where the depth is worth the longer start and end, or they
// fill the CUs once, and not where their last round is a nearly empty one.  64 rows a workgroup, inside layers of 2048 to 8192 tokens, us with one strip and with two, by K
// steps and n: 5: 136 6.8, 7.9, 224 8.0, 7.5, 256 8.3, 7.9, 280 11.2, 13.7, 512 13.7, 14.2.  9: 136 8.3, 8.6, 172 9.3, 9.6, 256 9.6, 8.9, 280 13.3, 16.0, 512 15.7,
// 15.9.  12: 136 9.0, 9.3, 172 9.6, 9.7, 256 10.4, 9.7, 280 14.1, 17.5, 512 17.0, 17.1.  16: 129 9.8, 9.5, 172 10.6, 10.0, 256 11.4, 10.0, 264 14.8, 17.8, 344
// 15.5, 18.5, 512 18.8, 17.8.  32: 129 14.0, 12.4, 172 14.9, 13.2, 256 16.2, 13.2, 264 20.7, 24.4, 344 23.1, 26.1, 512 30.4, 26.4.  With the weights in the
// caches, 32: 448 26.4, 26.3, 768 39.2, 41.3, 1056 56, 69; 64: 129 23.7, 20.0, 256 24.7, 19.7, 264 34.8, 40.8, 384 35.5, 37.5, 448 44.9, 38.2, 528 55, 61, 640
// 57.1, 56.9, 768 72.6, 62.6, 1024 99, 91, 1056 106, 108, 1600 168, 156.
bool stamp_hi6_two_strips(const stamp_plan* p, int own) {
  const int cus = stamp_device_cus(), kt = p->Kpad / BK;
  const int64_t groups = hi6_groups(p, own), n = hi6_strips(p) / 2 * groups, rounds = (n + cus - 1) / cus, last = n - (rounds - 1) * cus;
  if (hi6_np(p, own) != 2 || hi6_ng(p, own) != 1 || 2 * n <= cus) return false;  // (2 n up to cus: AHEAD)
  if (rounds == 1) return kt >= 16 || 8 * n >= 7 * cus;
  return kt >= 64 ? 2 * last > cus : kt >= 16 && rounds == 2 && 4 * last >= 3 * cus;
}

size_t stamp_hi6_bytes(const stamp_plan* p, int own) {
  const int M = hi6_rows(p, own), np = hi6_np(p, own), gr = 32 * np;
  return (size_t)((M + gr - 1) / gr) * (p->Kpad / 128) * (2 * np * kBlock6);
}

// Plans that this kernel serves.  Every workgroup reads its rows' and columns' whole depth from L2, so its time goes with
// the product M N d; the tiled int8 kernel shares operands through LDS and splits a tile's depth
// while it has few tiles: its time hardly grows until its tiles fill the CUs, but it needs a second launch (parts, top levels) or
// its longer start.  Layers with int8 against FP6, microseconds, with one strip of columns a workgroup throughout.  Without transform, all M rows at 8 bits: 512 x 4096 x 4096 40,
// 34, 1024 x 4096 x 4096 48, 57; 8192 x 1536 x 1536 75, 113; 2048 x 2048 x 2048 40, 45; 1024 x 2048 x 2048 36, 27; 4096 x
// 1024 x 1024 38, 35, 8192: 47, 62; 4096 x 4096 x 512 38, 55.  64 top rows a sequence, top levels: 2048 x 2048 x 4096 212 against 258 at
// depth 4096, 104 against 126 at depth 1024; 512 x 4096 x 4096 89, 76.  The lines fitted to 1364 such pairs (M 192 .. 16384,
// depth 192 .. 11008, d_out 16 .. 11008; five kinds of plan): M (d_out + 256) up to 6.5e6, and M (d_out + 768), the larger share of
// the rows' own operand, up to 8e5 + 8e9 / depth.  That is 0.3 % above always taking the better one on average and 22 % at worst,
// where a bound of 2e10 on the product is 6 % and 359 % (linear_forward_q of 7820 rows x 2656 x 12 27 us against 38).  With two strips
// (stamp_hi6_two_strips) 55 pairs around the line, 0.4 to 2.5 times it, are 2.2 % above the better one on average, 15 % at worst (3614 x
// 9344 -> 150 without transform, 2.0 times the line: 70, 61); 512 x 4096 x 4096 33.  The line stands where it was.
bool stamp_hi6_fits(const stamp_plan* p, int own) {
  const StampGeom& g = p->geom;
  const int M = hi6_rows(p, own);
  if (M < 1 || p->gen.group != 0) return false;
  if (!g.ident && !own && g.L > 0 && (g.k > 128 || (g.k & (g.k - 1)) != 0)) return false;  // whole sequences per workgroup
  const int choice = p->dbg[STAMP_CHOICE_HI_ROWS];
  if (choice != 0) return choice == 2;
  return M <= 128 || ((double)M * (g.N + 256) <= 6.5e6 && (double)M * (g.N + 768) <= 8.0e5 + 8.0e9 / g.d);
}

// Plans whose 4-bit rows' GEMM takes the 8-bit rows along: 128-row tiles (their kernel has the registers), whole blocks per tile and
// places for the rows above them (1-D, not below blocks of 16 tokens with many top levels), sums that fp32 holds exactly.
// Layers, us, rows' own kernel against this: 2048 x 11008 -> 4096 (3 levels) 93.6, 78.9; 2 x 1024 x 4096 -> 3 x 4096 140.5, 119; 3 x 777
// x 1184 -> 2305 35.7, 29.0; 512 x 1024 -> 1024 21.3, 17.1; 1024 x 2048 -> 2048, full depth 41.7, 34.7; 4096 x 2048 -> 1024 58.4, 56.4.
StampHiTiles stamp_hi_tiles(const stamp_plan* p, int own) {
  StampHiTiles t = {};
  const bool rag = p->rag.on;
  const StampGeom& g = rag ? p->bgeom : p->geom;
  if (p->gen.group != 0 || p->dbg[STAMP_CHOICE_HI_ROWS] != 0) return t;
  if (!rag && (p->gen.kind != kGenNone || g.ident || !p->fused_ok || p->unfused)) return t;
  const int rl = g.is2d ? 2 * g.r : g.r, khi = own || rag ? g.khi : g.k, L = rag ? 0 : g.L;
  if (rl < 3 || rl > 6 || khi < 1 || (g.is2d && L > 0) || g.d > 18720) return t;  // 128 * 7 * 18720 < 2^24
  const int lognb = 7 - rl, above = L > lognb ? L - lognb : 0;
  if ((1 << lognb) + above > kHiPlaces) return t;
  if (rag && p->rag.o && khi - 1 >= p->rag.nb) return t;  // no block left whose place the token left out could have
  const int M = rag ? (g.B * p->rag.nb) << p->rag.r : g.B * g.s;
  if (!stamp_gemm6_half_tiles(M, p->Npad)) return t;
  t.on = 1;
  t.lognb = lognb;
  t.k = rag ? p->rag.nb : g.k;
  t.khi = khi;
  t.L = L;
  t.o = rag ? p->rag.o : 0;
  return t;
}
size_t stamp_hi_tiles_bytes(const stamp_plan* p) {
  const size_t M = p->rag.on ? (size_t)(p->geom.B * p->rag.nb) << p->rag.r : (size_t)p->geom.B * p->geom.s;
  return (M + 127) / 128 * (p->Kpad / 128) * kBlock6;
}

StampHiOut stamp_hi6_out(const stamp_plan* p, uint8_t* a6, int own, const StampHiTiles& ht) {
  return StampHiOut{a6, hi6_np(p, own), own ? p->geom.khi : p->geom.k, ht};
}

StampHi6Pack stamp_hi6_pack(const stamp_plan* p, const int8_t* q_hi, uint8_t* a6, int own, const StampHiTiles& ht) {
  const StampGeom& g = p->geom;
  StampHi6Pack hp = {};
  hp.q_hi = q_hi;
  hp.out = stamp_hi6_out(p, a6, own, ht);
  hp.M = hi6_rows(p, own);
  hp.seq_rows = g.k;
  hp.d = g.d;
  hp.KT = p->Kpad / 128;
  hp.nseq = g.B;
  const int gr = 32 * hp.out.np;  // (the rows' own kernel reads whole groups)
  // A thread converts 32 channels (some 200 instructions), and a wave with a few of them takes as long as a full one: narrow layers
  // have threads for the rows (no top levels: each has one place), or for the places that can hold one, the first of a
  // tile.  Wide ones, where a place is whole waves, have them for all 16, which spreads those with work over more CUs.
  // linear_forward_q, us, all 16 places against these: blocks of 64, 4 x 1024 x 64 -> 1024 18.8, 12.4 (the rows' own kernel 15.3), 8 x
  // 1024 x 64 -> 256 16.8, 12.8; 16 x 200 x 128 -> 64, blocks of 16 16.5, 13.1.  Full depth, 16 against the 7 that can hold a row:
  // 8 x 4096 x 1024 -> 256 33.7, 34.6, 4 x 4096 x 2048 -> 512 36.4, 37.3.  With the present conversion, three layers of one quantized activation, 16 against
  // these: 4 x 1024 x 64 -> 1024 59.4, 55.3, 8 x 1024 x 64 -> 256 55.8, 56.3, 4 x 1024 x 480 -> 512, full depth 59.6, 60.9, 576 62.2, 63.9.
  const bool narrow = p->Kpad <= 512;
  hp.places = !narrow ? kHiPlaces : ht.L == 0 ? 0 : (1 << ht.lognb) + (ht.L > ht.lognb ? ht.L - ht.lognb : 0);
  const int rows = !ht.on ? (hp.M + gr - 1) / gr * gr : hp.places == 0 ? hp.M : ((g.B * ht.k + (1 << ht.lognb) - 1) >> ht.lognb) * hp.places;
  hp.threads = rows * hp.KT * 4;
  return hp;
}

hipError_t stamp_launch_hi6(const stamp_plan* p, const uint8_t* a6, const float* scales, int mode, void* out, int ld_out, int own,
                            void* Y, float norm, hipStream_t st) {
  Hi6Args h = {};
  h.a = stamp_gemm_args(p, scales, out);
  h.a.A = a6;
  h.a.Bq = p->qW6_dev;
  h.a.M = hi6_rows(p, own);
  h.a.ld_out = ld_out;
  if (own) h.a.g.k = p->geom.khi;  // the kernel sees a plan of khi top rows per sequence
  h.a.rag = p->rag;
  h.np = hi6_np(p, own);
  h.ng = hi6_ng(p, own);
  h.mode = mode;
  h.norm = norm;
  h.Y = Y;
  // workgroups up to one per CU: the rule of AHEAD
  if (hi6_strips(p) * hi6_groups(p, own) <= stamp_device_cus()) return h.np == 2 ? launch<2, false, true>(h, st) : launch<1, false, true>(h, st);
  if (stamp_hi6_two_strips(p, own)) return launch<2, false, false, 2>(h, st);
  return h.np == 1 ? launch<1, false, false>(h, st) : launch<2, false, false>(h, st);
}

// Without a limit on the rows: they are at most a 16th of the layer's tokens (one per 4 x 4 block), so this kernel stays the smaller
// part beside the 4-bit rows' GEMM.  The most of them, 16 x 4096 tokens with 256 each, 1152 -> 1152: linear_forward_q 178 us against
// 346 level by level; 64 x 4096, 640 -> 640: 312, 560.
hipError_t stamp_launch_hi6_grp(const stamp_plan* p, const uint8_t* h6, const float* sh, float* P, int own, hipStream_t st) {
  Hi6Args h = {};
  h.a = stamp_gemm_args(p, nullptr, P);
  h.a.A = h6;
  h.a.Bq = p->qWg6_dev;
  h.a.g = p->bgeom;
  if (own) h.a.g.k = p->bgeom.khi;
  h.a.M = h.a.g.B * h.a.g.k;
  h.a.ld_out = p->Npad;
  h.np = h.a.M <= 32 ? 1 : 2;
  h.ng = 1;
  h.norm = 1.0f;
  h.sa = sh;
  h.sw = p->swg6_dev;
  return h.np == 1 ? launch<1, true, false>(h, st) : launch<2, true, false>(h, st);
}
