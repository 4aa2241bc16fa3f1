// What the bottom kernels by lanes share (stamp_lanes1d.hip, stamp_lanes2d.hip): a lane holds 32 consecutive channels of its tokens.
#ifndef STAMP_LANES_H_
#define STAMP_LANES_H_
#include "stamp_bottom_kernel.h"

namespace {

using stamp_gemm::f16v;
using stamp_gemm::split_hi;
using stamp_gemm::store24;
using stamp_gemm::to_e2m3;
using stamp_gemm::u6v;

struct LaneArgs {
  const void* X;
  uint8_t* a6;       // operand of the 4-bit rows
  float* scales;
  float* abot;       // top levels: the block sums [B][s / 2^RLOG][d] go here, unfinished; else nullptr
  int s, d, k, khi, KT;
  int R;             // the plan's block length: 2^RLOG tokens are one of its parts
  size_t zeros_off;
  Hi6Out hi6;
  StampRag rag;
  int gb;            // row_off6
  int G, gridW;      // token grid: blocks per row, tokens per row
};

// Which of n units of ROWS rows a workgroup takes: 64 neighbouring rows go to one XCD.  The workgroups go to the eight XCDs in turn, and each
// of these has an L2 of its own, but rows 8 or 16 apart share every 16 bytes of the middle third of the operand, and units of fewer than
// eight rows share lines everywhere (row_off6): unit by unit they were put together from several L2s.  Rows without transform, us, before
// and with this: 8192 x 4096 bf16 20.2, 17.6, 32768 x 4096 77.8, 65.0, 8192 x 11008 62.8, 49.5 (2 rows a unit), 8192 x 4096 fp32 32.2, 30.0; Haar blocks
// of 8: 8192 x 4096 23.1, 20.5, 16384 x 4096 41.7, 36.3, of 16: 49.7, 48.0.  (Rows that share those 16 bytes in one workgroup, four rows of
// eight each, instead: 22.3 and 91.8 for the first two.)
template <int ROWS>
__device__ __forceinline__ int unit_of_block(int blk, int n) {
  constexpr int U = 64 / ROWS;
  return blk < n / (8 * U) * (8 * U) ? (blk & ~(8 * U - 1)) + (blk & 7) * U + ((blk >> 3) & (U - 1)) : blk;
}

// codes of 8-bit rows, 16 h + l, as two fragments
__device__ __forceinline__ void store_hi24(const Hi6Out& o, int m, int KT, f16v ev, f16v od, int c) {
  u6v h, l;
  split_hi(ev, od, h, l);
  const uint32_t off = chan_off6((uint32_t)c, hi_step_bytes(o));
  hi_rows(o, m, KT, [&](uint8_t* dst, bool hh, int lo, bool lh) {
    store24(dst + off, h, hh);
    store24(dst + off + lo, l, lh);
  });
}

// the sum of this lane's partner at lane distance 2^(l - 2)
template <int l>
__device__ __forceinline__ float partner(float x) {
  const int i = __float_as_int(x);
  if constexpr (l == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, true));       // quad_perm [1,0,3,2]
  else if constexpr (l == 3) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, true));  // quad_perm [2,3,0,1]
  else {
    static_assert(l == 4, "");
    const int lo = __builtin_amdgcn_update_dpp(0, i, 0x104, 0xF, 0xF, true);             // row_shl 4: lane n takes lane n + 4
    return __int_as_float(__builtin_amdgcn_update_dpp(lo, i, 0x114, 0xF, 0xA, false));   // row_shr 4 into the odd quads
  }
}

// largest over the lanes of equal token pair (NL lanes apart)
template <int NL>
__device__ __forceinline__ uint32_t across_groups(uint32_t x) {
  if constexpr (NL <= 1) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, true));  // row_ror 1
  if constexpr (NL <= 2) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, true));  // row_ror 2
  if constexpr (NL <= 4) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true));  // row_ror 4
  if constexpr (NL <= 8) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true));  // row_ror 8
  auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = max(p[0], p[1]);
  auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return max(q[0], q[1]);
}

// largest magnitude (ASYM: order key of the largest value) of 32 channels.  A NaN is passed over unless it has eight
// neighbours of its kind (one thread's share in the streaming kernels); nan_max: it is the largest value.
template <bool ASYM>
struct RowMax {
  float hi[4], lo[4], nan = 0.0f;  // nan: not 0 if a value is no number or infinite
  template <bool NANMAX>
  __device__ __forceinline__ void add(int c, float v) {
    const float x = ASYM ? v : fabsf(v);
    hi[c >> 3] = (c & 7) == 0 ? x : fmaxf(hi[c >> 3], x);
    if constexpr (ASYM) lo[c >> 3] = (c & 7) == 0 ? x : fminf(lo[c >> 3], x);
    if constexpr (NANMAX) nan = __builtin_fmaf(v, 0.0f, nan);
  }
  __device__ __forceinline__ uint32_t pos() const {
    uint32_t m = 0u;
#pragma unroll
    for (int g = 0; g < 4; ++g) m = max(m, ASYM ? fkey(hi[g]) : __float_as_uint(hi[g]));
    return m;
  }
  __device__ __forceinline__ uint32_t neg() const {
    uint32_t m = 0u;
#pragma unroll
    for (int g = 0; g < 4; ++g) m = max(m, fkey(-lo[g]));
    return m;
  }
};

// scale, reciprocal and offset of a row from its maxima (already times the row's norm)
template <bool ASYM>
__device__ __forceinline__ void row_params(float hi, float nlo, float qmax, float& scale, float& inv, float& z) {
  scale = inv = z = 0.0f;
  if constexpr (ASYM) {
    asym_params(hi, nlo, qmax, scale, inv, z);
  } else if (hi > 0.0f) {
    scale = __fdiv_rn(hi, qmax);
    inv = __fdiv_rn(qmax, hi);
  }
}

// largest over the waves of one row's maxima
__device__ __forceinline__ uint32_t max_of_waves(const uint32_t (&part)[16], int nw) {
  const u4* q = reinterpret_cast<const u4*>(&part[0]);
  uint32_t mx = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u4 v = q[i];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (4 * i + w < nw) mx = max(mx, v[w]);
  }
  return mx;
}

}  // namespace

#endif  // STAMP_LANES_H_
