// Internal declarations shared by the HIP sources of the STaMP library (gfx950 only).
#ifndef STAMP_INTERNAL_H_
#define STAMP_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "stamp.h"

#define STAMP_HD __host__ __device__ __forceinline__

// ---------------------------------------------------------------------------------------------
// Geometry of a plan.  The J-level transform is split at level r = log2(seq_len / k_hi) (1-D) or
// log4 (2-D): the "bottom" r levels act inside aligned blocks of R tokens and produce the R-1
// 4-bit rows of each block; the "top" J-r levels act on the k_hi block sums and produce the k_hi
// 8-bit rows.
// ---------------------------------------------------------------------------------------------
struct StampGeom {
  int32_t B, s, d, N;
  int32_t is2d;      // 0: 1-D stream, 1: 2-D grid
  int32_t J;         // total levels of the transform (plan argument)
  int32_t L;         // top levels J - r: levels applied to the k block sums (0 = the block sums themselves)
  int32_t r;         // bottom levels (inside a block)
  int32_t R;         // tokens per block: 2^r (1-D) or 4^r (2-D)
  int32_t k;         // number of blocks per sequence = rows of the top part (held as int8 codes, q_hi)
  int32_t khi;       // how many of them are 8-bit rows (k_hi); the others carry 4-bit codes (J < log2(seq_len / k_hi))
  int32_t G;         // 2-D: blocks per grid side (k = G*G); 1-D: unused (0)
  int32_t g;         // 2-D: tokens per block side (2^r); 1-D: unused (0)
  int32_t gridW;     // 2-D: tokens per grid row
  int32_t x_bf16;    // input dtype is bf16
  int32_t y_bf16;    // output dtype is bf16
  int32_t asym;      // asymmetric activation codes: stored code - 2^(b-1), offsets z next to the scales
  int32_t ident;     // no sequence transform: tokens 0..k-1 are the 8-bit rows, physical row = token (J = r = 0, R = 1)
                     // (also set for plans of the general path, whose quantizer and GEMM see transformed tokens as rows)
};

// General path: the transform runs level by level over fp32 buffers in the workspace (stamp_general.hip).
enum StampGenKind { kGenNone = 0, kGenCopy, kGenHaarRagged, kGenHaarClassic, kGenHaar2d, kGenWht, kGenDct };
struct StampGen {
  int32_t kind;        // StampGenKind
  int32_t levels;
  int32_t skip;        // first token left out (ragged Haar)
  int32_t group;       // 0 or 64
  int32_t bias_mode;   // 1: transformed bias
  int32_t gridH, gridW;
};

// Blocked form of a 1-D Haar transform of any length, optionally with the first token left out (o = 1): the n = s - o
// transformed tokens are nb blocks of R = 2^r tokens, r = the number of levels, the last one of mlast <= R tokens; a
// block's coefficients are one approximation and R - 1 details (fewer in a short block), as in the power-of-two case.
// Block order: row b * nb * R + j * R + e, e = in-block position (0 = the approximation).
struct StampRag {
  int32_t on, o, n, nb, mlast, r;
};
// The 8-bit rows in the tiles of the 4-bit rows' GEMM (128 rows of 2^lognb blocks): a tile's outputs need the sums of its own
// blocks, hence their 8-bit rows and, with top levels, the rows above them in the tree.  Every tile has 16 places for such rows: its
// blocks' rows where the in-place network of the top levels leaves them, then one place per level above the tile's
// sub-tree, finest first.  A row that several tiles need is stored for each.
struct StampHiTiles {
  int32_t on, lognb;
  int32_t k, khi;    // blocks per sequence, 8-bit rows per sequence
  int32_t L, o;      // top levels; 1: the token left out is 8-bit row 0 (its place: that of the first block with a 4-bit sum)
};
constexpr int kHiPlaces = 16;
// 8-bit row `slot` of sequence b: its place in the tiles tile .. tile + ntiles - 1
STAMP_HD void stamp_hi_places(const StampHiTiles& t, int b, int slot, int* tile, int* ntiles, int* place) {
  const int nb = 1 << t.lognb;
  *ntiles = 1;
  if (t.L == 0) {
    const int j = t.o ? (slot == 0 ? t.khi - 1 : slot - 1) : slot, g = b * t.k + j;
    *tile = g >> t.lognb;
    *place = g & (nb - 1);
    return;
  }
  const bool apx = slot < (t.k >> t.L);
  const int m = apx ? 0 : 31 - __builtin_clz((unsigned)slot);
  const int lev = apx ? t.L : 31 - __builtin_clz((unsigned)t.k) - m, i = apx ? slot : slot - (1 << m);
  const int g = b * t.k + (i << lev);  // the first of the row's 2^lev blocks
  *tile = g >> t.lognb;
  if (lev <= t.lognb) {
    *place = (g & (nb - 1)) + (apx ? 0 : 1 << (lev - 1));
  } else {
    *ntiles = 1 << (lev - t.lognb);
    *place = apx ? 0 : nb + lev - t.lognb - 1;
  }
}

// The other way round: the row (of sequence *b, its level within the top part: *up) at a tile's place, -1: none
STAMP_HD int stamp_hi_slot_of_place(const StampHiTiles& t, int nseq, int tile, int p, int* b, int* up) {
  const int nb = 1 << t.lognb, g = (tile << t.lognb) + (p < nb ? p : 0);
  *b = g / t.k;
  *up = 0;
  const int j = g - *b * t.k;
  if (*b >= nseq) return -1;
  if (t.L == 0) {
    if (p >= nb || j >= t.khi) return -1;
    return t.o ? (j == t.khi - 1 ? 0 : j + 1) : j;
  }
  const int lev = p < nb ? (j == 0 ? 32 : __builtin_ctz((unsigned)j)) + 1 : t.lognb + 1 + p - nb;
  if (p >= nb && lev > t.L) return -1;
  // place 0 of a tile below the tree's top: its approximation
  if (p < nb && (lev > t.L || (p == 0 && t.lognb < t.L))) {
    *up = t.L;
    return j >> t.L;
  }
  *up = lev;
  return (t.k >> lev) + (j >> lev);
}

// STaMP slot of in-block position e of block j, -1 where a short block has no such coefficient.  The details of level l
// sit from slot o + ceil(n / 2^l) on; one exists where both of its halves do.
STAMP_HD int stamp_rag_slot(const StampRag& q, int j, int e) {
  if (e == 0) return q.o + j;
  const int m = 31 - __builtin_clz((unsigned)e), l = q.r - m, idx = (j << m) + e - (1 << m);
  if (2 * idx + 1 >= ((q.n + (1 << (l - 1)) - 1) >> (l - 1))) return -1;
  return q.o + ((q.n + (1 << l) - 1) >> l) + idx;
}
// How often a node of level l (index i inside the short last block of m tokens) is carried up unchanged on its way to
// level r: where a level has an odd number of nodes, the last one has no partner.
STAMP_HD int stamp_rag_carries(int m, int l, int i, int r) {
  int cnt = 0;
  for (int k = l; k < r; ++k) {
    const int nk = (m + (1 << k) - 1) >> k;
    cnt += (i == nk - 1 && (nk & 1)) ? 1 : 0;
    i >>= 1;
  }
  return cnt;
}

// Position inside a block ("e", 0 = the block sum, e >= 1 the in-block detail rows in STaMP
// order) of the coefficient that the in-place butterfly network leaves at natural position q.
// 1-D: in-place butterflies at stride 2^l leave the level-l difference of pair i at position
// i*2^l + 2^(l-1).
STAMP_HD int stamp_e_of_natural_1d(int q, int n /* block length, power of two */) {
  if (q == 0) return 0;
  int t = __builtin_ctz((unsigned)q);  // level - 1
  return (n >> (t + 1)) + (q >> (t + 1));
}

// 2-D: natural position (y, x) in a g x g block; the in-place network leaves at
// (2^l i + dy 2^(l-1), 2^l j + dx 2^(l-1)) the band (dy, dx) of level l: (0,1) = difference along
// the width, (1,0) = along the height, (1,1) = diagonal.
STAMP_HD int stamp_e_of_natural_2d(int y, int x, int g) {
  if (y == 0 && x == 0) return 0;
  int t = __builtin_ctz((unsigned)(y | x));  // level - 1
  int by = (y >> t) & 1, bx = (x >> t) & 1;
  int band = by ? (bx ? 2 : 1) : 0;          // W, H, D
  int gl = g >> (t + 1);                     // side of each band of that level
  return gl * gl * (1 + band) + (y >> (t + 1)) * gl + (x >> (t + 1));
}

// Top part, L levels over n block sums (1-D) / G x G block sums (2-D): STaMP slot (< n, < G*G) of the
// coefficient that L in-place butterfly levels leave at natural position q / (y, x), and its level counted
// within the top part (L for the remaining approximations, which come first in STaMP order).
STAMP_HD int stamp_top_slot_1d(int q, int n, int L, int* lvl_top) {
  const int t = (q == 0) ? 32 : __builtin_ctz((unsigned)q);
  if (t >= L) { *lvl_top = L; return q >> L; }
  *lvl_top = t + 1;
  return (n >> (t + 1)) + (q >> (t + 1));
}
STAMP_HD int stamp_top_slot_2d(int y, int x, int G, int L, int* lvl_top) {
  const int t = ((y | x) == 0) ? 32 : __builtin_ctz((unsigned)(y | x));
  if (t >= L) { *lvl_top = L; return (y >> L) * (G >> L) + (x >> L); }
  *lvl_top = t + 1;
  return stamp_e_of_natural_2d(y, x, G);
}
// Level (counted over the whole transform) of the 8-bit STaMP slot p.
STAMP_HD int stamp_level_of_top_slot(int p, int k, int G, int is2d, int r, int L) {
  if (!is2d) {
    if (p < (k >> L)) return r + L;
    return r + (31 - __builtin_clz((unsigned)k)) - (31 - __builtin_clz((unsigned)p));
  }
  if (p < (G >> L) * (G >> L)) return r + L;
  return r + (31 - __builtin_clz((unsigned)G)) - ((31 - __builtin_clz((unsigned)p)) >> 1);
}

// STaMP slot p (whole sequence) of in-block position e >= 1 of block j.
// 1-D: e = 2^m + i  ->  p = (k + j) * 2^m + i.
STAMP_HD int stamp_slot_of_block_e_1d(int j, int e, int k) {
  int m = 31 - __builtin_clz((unsigned)e);
  return ((k + j) << m) + (e - (1 << m));
}

// 2-D: block (bi, bj) of a G x G block grid, e = gl^2 (1 + band) + yy gl + xx  ->
// p = (G gl)^2 (1 + band) + (bi gl + yy)(G gl) + bj gl + xx.
STAMP_HD int stamp_slot_of_block_e_2d(int bi, int bj, int e, int G) {
  int m = (31 - __builtin_clz((unsigned)e)) >> 1;  // gl = 2^m, since gl^2 <= e < 4 gl^2
  int gl = 1 << m;
  int band = (e >> (2 * m)) - 1;
  int rem = e - ((1 + band) << (2 * m));
  int yy = rem >> m, xx = rem & (gl - 1);
  int Gl = G * gl;
  return Gl * Gl * (1 + band) + (bi * gl + yy) * Gl + bj * gl + xx;
}

// Level (1 = finest) of in-block position e >= 1 in a block of R tokens.
STAMP_HD int stamp_level_of_e_1d(int e, int r) { return r - (31 - __builtin_clz((unsigned)e)); }
STAMP_HD int stamp_level_of_e_2d(int e, int r) { return r - ((31 - __builtin_clz((unsigned)e)) >> 1); }

// Byte offset of (output column n, permuted channel position c) in the stored weight:
// [Npad/128][Kpad/128][128 columns][128 positions].
STAMP_HD size_t stamp_w_offset(int n, int c, int Kpad) {
  return (((size_t)(n >> 7) * (size_t)(Kpad >> 7) + (size_t)(c >> 7)) * 128 + (size_t)(n & 127)) * 128 + (size_t)(c & 127);
}

// Byte offset of (physical row m over all sequences, channel c) in the tiled 4-bit activation:
// [Mpad/256][Kpad/128][256 rows][64 bytes], two channels per byte.
STAMP_HD size_t stamp_qlo_offset(size_t m, int c, int Kpad) {
  return (((m >> 8) * (size_t)(Kpad >> 7) + (size_t)(c >> 7)) * 256 + (m & 255)) * 64 + (size_t)((c & 127) >> 1);
}

// ---------------------------------------------------------------------------------------------
// The plan.
// ---------------------------------------------------------------------------------------------
struct stamp_plan {
  stamp_plan_desc_t desc;
  StampGeom geom;
  int32_t Kpad, Npad;       // GEMM-padded depth and width of the stored weight
  int32_t Mpad;             // batch * seq_len rounded up to the GEMM's 256-row tile
  int8_t* qW_dev;           // tiled int8 weight codes * 16 (see stamp_w_offset), K order permuted per 16 channels (not with per-block scales)
  float* sw_dev;            // [Npad] weight scales (0 beyond d_out, and with per-block scales)
  float* bias_dev;          // [Npad] bias or nullptr
  float* colsum_dev;        // [Npad] sum over input channels of the weight codes (exact integers as fp32)
  int32_t* row_of_coeff;    // host, [s]
  uint8_t* qW6_dev;         // the same weight codes as E2M3 numbers in the operand layout of the FP6 GEMM
  int32_t engine;           // matrix pipeline of the 4-bit rows' GEMM: STAMP_GEMM_INT8 or STAMP_GEMM_FP6
  int32_t hi_ksplit;        // parts the depth of the 8-bit rows' GEMM is split into (partial rows in the workspace)
  int32_t hi_ksplit_own;    // the same when only the first khi top rows go through that GEMM (stamp_own_top)
  int32_t unfused;          // 1: separate inverse kernel
  int32_t fused_ok;         // shape allows the fused epilogue
  StampGen gen;             // general path (kind != kGenNone)
  StampRag rag;             // general path, 1-D Haar of any length: blocked form (rag.on), geometry in bgeom
  StampGeom bgeom;
  int32_t* perm_dev;        // general path, WHT in several passes: [s] STaMP slot of every row of the Hadamard-ordered result
  float* ell_dev;           // general path, transformed bias: [s] l = L 1
  double* dct_dev;          // general path, DCT: [s][s] orthonormal DCT-II matrix
  int8_t* qWg_dev;          // per-block scales: weight codes [Npad128][d_in] int8
  float* swg_dev;           // per-block scales: [d_in / 64][Npad128]
  // per-block scales on the blocked 2-D Haar transform (stamp_grouped.hip), geometry in bgeom: quantizer, GEMM with inverse
  int32_t grp_quant, grp;
  uint8_t* qWg6_dev;        // its weights as FP6 operand and their scales
  float* swg6_dev;
  size_t ws_grp[4];         // its scratch (over ws_T, ws_Yt)
  size_t ws_T[3], ws_Yt[3], ws_codes8, ws_scalesg;  // general path workspace (byte offsets)
  // the 8-bit rows through the kernel for few rows (stamp_hi6.hip), [1]: only the first khi rows of every sequence
  int32_t hi6[2];
  size_t ws_hi6;            // their operand
  // the same where blocks are quantized in parts of 8 tokens, 0: they are not; in which form (the layout's room is for that one)
  size_t ws_parts_hi;
  StampHiTiles parts_tiles;
  int32_t direct_ok;        // the quantizer may write the FP6 operands itself (the 8-bit rows' over ws_qhi)
  int32_t dbg[STAMP_CHOICE_COUNT];  // stamp_debug_set_choice: 0 by rule, 1 / 2 the one or the other form
  size_t ws_ba6, ws_bP;     // blocked form: the 4-bit rows in block order (over ws_T), the block sums (over ws_Yt)
  // workspace layout (byte offsets, 256-aligned)
  size_t ws_abot, ws_rowmax, ws_gpart, ws_qhi, ws_qlo, ws_scales, ws_ythi, ws_P, ws_a6, ws_ytlo, ws_total;
  size_t ws_base;           // ws_total without an 8-bit operand behind everything else
};

// Dynamic-LDS limit of a kernel, raised once per device and kernel (the attribute belongs to the device's
// copy of the function): `done` is the kernel's own table, one size per device.
constexpr int kStampMaxDevices = 64;
inline std::mutex& stamp_lds_mutex() {
  static std::mutex m;  // one lock for all tables: taken once per launch, never contended for long
  return m;
}
inline hipError_t stamp_allow_lds(const void* kernel, size_t bytes, size_t (&done)[kStampMaxDevices]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kStampMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(stamp_lds_mutex());  // plans may be used from several host threads
  if (bytes <= done[dev]) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done[dev] = bytes;
  return e;
}

// compute units of the device that is current at the first call
int stamp_device_cus();

// ---- launchers implemented in the kernel files (all asynchronous on `st`) ----
hipError_t stamp_launch_weight_quant(const stamp_plan* p, const float* W, hipStream_t st, uint32_t* colmax_tmp);
// part: 1 = bottom kernel only, 2 = top + 8-bit rows only, 3 = both
// scales: [B*s] scales, followed by [B*s] offsets z for asymmetric plans
// gpart: [2][nsplit][B*s] partial row maxima when the channels are split over workgroups (nsplit > 1), else unused
int stamp_actquant_nsplit(const stamp_plan* p);
// plans without top levels: the bottom kernel also quantizes the block sums (no k_top, no k_quant_hi)
bool stamp_top_in_bottom(const stamp_plan* p);
// packed codes of 8 x 8 blocks whose four sub-blocks one workgroup takes side by side (k_bottom2d_quads: up to 1536 channels by its threads;
// up to two blocks per CU: with more the CUs are full either way)
bool stamp_bottom_quads(const stamp_plan* p);
// dir: the codes leave as FP6 operands (4-bit rows, 8-bit rows) instead of in q_hi / q_lo, which are not written
// The FP6 operand of the 8-bit rows: for the kernel of their own (stamp_hi6.h; np, rows m), or in the places of the 4-bit rows'
// tiles (ht.on).
struct StampHiOut {
  uint8_t* p;    // nullptr: none
  int32_t np;
  int32_t seq;   // 8-bit rows per sequence: row m is row m % seq of sequence m / seq
  StampHiTiles ht;
};
struct StampDirect {
  uint8_t* a6;
  StampHiOut hi;
  int32_t lo_packed;  // the 4-bit rows do leave in q_lo, and the top levels' launch converts them
  int32_t parts;      // longer blocks in parts of 8 tokens (abot: [B][s / 8][d])
};
hipError_t stamp_launch_actquant(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo,
                                 float* scales, float* abot, uint32_t* rowmax, uint32_t* gpart, hipStream_t st, int part = 3,
                                 const StampDirect* dir = nullptr);
// mode: 0 = int32 accumulators in STaMP row order (debug), 1 = dequantized fp32 rows (hi -> Yt_hi
// [hi_ksplit][B*k, N] partial rows, lo -> Yt_lo [B*s, N] physical rows), 2 = lo rows with fused in-block inverse -> Y,
// 3 = lo rows of an identity plan: dequantized + bias -> Y.
bool stamp_hi_wide_tiles(int M, int Npad);
int stamp_hi_ksplit(const stamp_plan* p, int rows_per_seq);
// ld_out > 0 (mode 1): row stride of `out` in floats instead of d_out
// first_khi_only (mode 1): only the first khi rows of every sequence are multiplied, depth split into
// hi_ksplit_own parts, rows of `out` numbered b * khi + p
hipError_t stamp_launch_gemm_hi(const stamp_plan* p, const int8_t* q_hi, const float* scales, int mode,
                                void* out, hipStream_t st, int ld_out = 0, bool first_khi_only = false);
// P[row][0..ncols) = sum over the parts of src[part][row][0..ncols), rows < nrows
hipError_t stamp_launch_sum_parts(const float* src, int nparts, int nrows, int ncols, float* P, int ldP, hipStream_t st);
bool stamp_hi_rows_are_block_sums(const stamp_plan* p);
// mode 2 of stamp_launch_gemm_hi is available: dequantization + top levels of the inverse in the GEMM's tiles, out = P
bool stamp_hi_top_fused(const stamp_plan* p);
hipError_t stamp_launch_gemm_lo(const stamp_plan* p, const uint8_t* q_lo, const float* scales, int mode,
                                void* out, const float* P, hipStream_t st);
// FP6 engine of the 4-bit rows: operand sizes, plan-time weight codes (colmax: bit patterns of the column
// maxima, as left by stamp_launch_weight_quant), conversion of the packed 4-bit rows, and the GEMM (modes as above).
size_t stamp_a6_bytes(const stamp_plan* p);
size_t stamp_b6_bytes(const stamp_plan* p);
hipError_t stamp_launch_weight_quant6(const stamp_plan* p, const float* W, const uint32_t* colmax, hipStream_t st);
// hi: 8-bit rows to convert in the same launch (nullptr: none); q_lo may be nullptr then
struct StampHi6Pack {
  const int8_t* q_hi;
  StampHiOut out;
  int32_t M, seq_rows, nseq, d, KT, threads;  // rows, rows a sequence has in q_hi (it uses out.seq)
  int32_t places;                             // of a tile that threads are launched for; 0: threads for the rows
};
hipError_t stamp_launch_repack6(const stamp_plan* p, const uint8_t* q_lo, uint8_t* a6, hipStream_t st, const StampHi6Pack* hi = nullptr);
// the 8-bit rows' GEMM on the FP6 pipeline (few rows), own: only the first khi rows of every sequence.  mode 0: block sums
// -> out [M][ld_out] (top levels of the inverse included), 1: rows + bias -> Y (plans without transform), 2: rows -> fp32
// [B*s][N] in STaMP order, 3: blocked form: block sums times norm -> out, the token left out + bias -> Y
bool stamp_hi6_fits(const stamp_plan* p, int own);
size_t stamp_hi6_bytes(const stamp_plan* p, int own);
int stamp_hi6_rows_per_workgroup(const stamp_plan* p, int own);
bool stamp_hi6_two_strips(const stamp_plan* p, int own);
// the operand at `a6`; ht: in the tiles' places instead
StampHiOut stamp_hi6_out(const stamp_plan* p, uint8_t* a6, int own, const StampHiTiles& ht);
StampHi6Pack stamp_hi6_pack(const stamp_plan* p, const int8_t* q_hi, uint8_t* a6, int own, const StampHiTiles& ht);
// whether the 4-bit rows' GEMM (FP6 engine: the layout does not depend on the engine, callers ask for it) takes the 8-bit
// rows along (ht.on), and the bytes of their operand
StampHiTiles stamp_hi_tiles(const stamp_plan* p, int own);
size_t stamp_hi_tiles_bytes(const stamp_plan* p);
hipError_t stamp_launch_hi6(const stamp_plan* p, const uint8_t* a6, const float* scales, int mode, void* out, int ld_out, int own,
                            void* Y, float norm, hipStream_t st);
// blocked form (p->rag.on): the same conversion from rows in STaMP order to block order; packed nibbles in block order
// for the int8 engine; and the two GEMMs with the inverse transform in their epilogue
size_t stamp_rag_a6_bytes(const stamp_plan* p);
hipError_t stamp_launch_repack6_rag(const stamp_plan* p, const uint8_t* q_lo, uint8_t* a6, hipStream_t st, const StampHi6Pack* hi);
hipError_t stamp_launch_gather_lo_rag(const stamp_plan* p, const uint8_t* q_lo, uint8_t* q_blk, hipStream_t st);
// hi (ht.on): the 8-bit rows' operand in the tiles' places, P is not read then
hipError_t stamp_launch_gemm_lo6_rag(const stamp_plan* p, const uint8_t* a6, const float* scales, void* Y, const float* P, hipStream_t st,
                                     const StampHiOut* hi = nullptr);
hipError_t stamp_launch_gemm_lo_rag(const stamp_plan* p, const uint8_t* q_blk, const float* scales, void* Y, const float* P, hipStream_t st);
// 8-bit rows' partial rows [nparts][B*khi][N] -> block sums P [B*khi][Npad] (times the blocks' norm); with the first
// token left out, its row (+ bias) -> Y
hipError_t stamp_launch_rag_top(const stamp_plan* p, const float* ythi, int nparts, float* P, void* Y, hipStream_t st);
// own_top (mode 2, plans without top levels): the blocks from khi on take their sum from their own coefficient 0,
// a 4-bit row of a6 like any other (the quantizer writes it there as well), and P holds khi rows per sequence
hipError_t stamp_launch_gemm_lo6(const stamp_plan* p, const uint8_t* a6, const float* scales, int mode, void* out,
                                 const float* P, hipStream_t st, int own_top = 0, const StampHiOut* hi = nullptr);
// 4-bit rows of the FP6 engine (row_off6): log2 of the rows that the fused epilogue keeps in a lane, 2 where rows are tokens
inline int stamp_row_group_bit(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  const int rl = g.ident ? 2 : g.is2d ? 2 * g.r : g.r;
  return rl < 2 ? 2 : rl > 6 ? 6 : rl;
}
// whether the FP6 GEMM over M rows takes 128 x 256 tiles
bool stamp_gemm6_half_tiles(int M, int Npad);
bool stamp_gemm6_pairs(int M, int Npad, int Kpad, int mode);  // two workgroups of 128 x 256 tiles per CU
// identity plans: 8-bit rows' dequantized partial rows [nparts][B*k][N] (+ bias) -> Y rows of tokens 0..k-1
hipError_t stamp_launch_hi_rows_out(const stamp_plan* p, const float* Yt_hi, void* Y, hipStream_t st, int nparts);
// P: block sums [B*k][ldP]; nparts partial sources (each B*k*ncols floats apart) are added while reading
hipError_t stamp_launch_inverse_top(const stamp_plan* p, const float* Yt_hi, int hi_row_stride_is_stamp,
                                    int ncols, float* P, int ldP, hipStream_t st, int nparts = 1);
hipError_t stamp_launch_inverse_bottom(const stamp_plan* p, const float* Yt_lo, int src_is_stamp_order,
                                       const float* P, int ldP, int ncols, const float* bias, void* Y, hipStream_t st);

// ---- general path (stamp_general.hip) ----
float stamp_haar_norm_host(int level);  // fl(2^(-level/2))
hipError_t stamp_gen_plan_tables(stamp_plan* p, const float* W, hipStream_t st);  // device tables and grouped weights
void stamp_gen_plan_free(stamp_plan* p);
// X -> transformed tokens T [B, s, d] fp32 in STaMP order; returns the buffer that holds T (one of the three)
hipError_t stamp_gen_forward(const stamp_plan* p, const void* X, float* const (&buf)[3], float** T_out, hipStream_t st);
// Yt [B, s, ncols] fp32 in STaMP order (buf[0], only read) -> Y; buf[1], buf[2]: the levels' work buffers
hipError_t stamp_gen_inverse(const stamp_plan* p, float* const (&buf)[3], int ncols, const float* bias, void* Y, hipStream_t st);
// Bottom kernels that leave FP6 operands (stamp_lanes1d.hip): blocks of 2^rlog tokens (3, 4), or parts of longer ones with their
// sums left in abot.
bool stamp_lanes1d_fits(const stamp_plan* p, int rlog);
hipError_t stamp_launch_lanes1d(const stamp_plan* p, int rlog, const void* X, uint8_t* a6, float* scales, float* abot, const StampHiOut& hi,
                                hipStream_t st);
// the same for 4 x 4 and 8 x 8 blocks of a token grid
bool stamp_lanes2d_fits(const stamp_plan* p);
hipError_t stamp_launch_lanes2d(const stamp_plan* p, const void* X, uint8_t* a6, float* scales, float* abot, const StampHiOut& hi, hipStream_t st);
// rows as they are (k = the first 8-bit rows of every sequence) -> operands and scales
hipError_t stamp_launch_lanes_rows(const stamp_plan* p, const void* X, int x_bf16, uint8_t* a6, float* scales, const StampHiOut& hi, hipStream_t st);
// the levels above parts of 8 tokens: their sums [B][s / 8][d] (overwritten) -> operands and scales of these rows
hipError_t stamp_launch_top_parts(const stamp_plan* p, float* abot, uint8_t* a6, float* scales, const StampHiOut& hi, hipStream_t st);
// DCT of a power-of-two length with the points in registers (stamp_dct.hip): plans it takes, and src -> T (inv = 0), src -> Y (+ bias)
bool stamp_dct_in_registers(int s, int B, int ld);
hipError_t stamp_launch_dct_reg(const stamp_plan* p, int inv, const void* src, int in_kind, float* T, void* Y, const float* bias, int ld,
                                hipStream_t st);
// blocked form: X -> codes and scales in STaMP order in one pass; false where the kernel does not take the plan or X
bool stamp_rag_quantizes(const stamp_plan* p, const void* X);
hipError_t stamp_launch_actquant_rag(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, hipStream_t st,
                                     const StampDirect* dir = nullptr);
hipError_t stamp_launch_quant_rows_f32(const stamp_plan* p, const float* T, int8_t* q_hi, uint8_t* q_lo, float* scales, hipStream_t st,
                                       const StampDirect* dir = nullptr);
hipError_t stamp_launch_quant_rows_grouped(const stamp_plan* p, const float* T, int8_t* codes, float* scales, hipStream_t st);
// per-block scales, blocked 2-D Haar (p->grp): X -> codes and scales in STaMP order (abot: [B*k][d] fp32 scratch), and from
// there to Y
void stamp_grp_bytes(const stamp_plan* p, size_t (&n)[4]);
hipError_t stamp_grp_plan_weights(stamp_plan* p, hipStream_t st);
hipError_t stamp_launch_grp_quant(const stamp_plan* p, const void* X, int8_t* codes, float* scales, float* abot, hipStream_t st);
hipError_t stamp_launch_grp_forward(const stamp_plan* p, const int8_t* codes, const float* scales, uint8_t* const (&buf)[4], float* P, void* Y,
                                    hipStream_t st);
hipError_t stamp_launch_hi6_grp(const stamp_plan* p, const uint8_t* h6, const float* sh, float* P, int own, hipStream_t st);
hipError_t stamp_launch_gemm_grouped(const stamp_plan* p, const int8_t* codes, const float* scales, float* Yt, hipStream_t st);
hipError_t stamp_launch_bf16_to_f32(const void* src, float* dst, size_t n, hipStream_t st);
hipError_t stamp_launch_merge_hi(const stamp_plan* p, const float* ythi, int nparts, float* Yt, hipStream_t st);
hipError_t stamp_launch_add_ell_bias(const stamp_plan* p, float* Yt, hipStream_t st);

#endif  // STAMP_INTERNAL_H_
