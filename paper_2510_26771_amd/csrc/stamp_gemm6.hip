// GEMM of the 4-bit rows of the STaMP linear layer on the FP6 matrix pipeline of gfx950 (step
// "Y <- X W" of Algorithm "STaMP Linear" for the rows quantized to 4 bits against 4-bit weights).
//
// A 4-bit code c in [-8, 7] is held as the E2M3 number c / 8: for |c| < 8 sign bit, exponent field 0,
// mantissa field |c| (a subnormal); |c| = 8 is 1.0 (exponent field 1, mantissa 0): either way the six
// bits are just sign and 4-bit magnitude.  v_mfma_f32_32x32x64_f8f6f4
// multiplies such operands exactly and accumulates in fp32; every product is a multiple of 1/64 and a
// whole sum stays below 2^24 / 64 in magnitude (|c c'| <= 56 and d_in <= 32768: 56 * 32768 < 2^24), so the fp32 accumulator
// holds acc / 64 EXACTLY, where acc is the integer sum the int8 pipeline computes: same result bit for
// bit, at twice the matrix rate per clock.  The factor 64 is folded into the row scale.
//
// The products are v_mfma_f32_16x16x128_f8f6f4: as many operations per clock as the 32 x 32 x 64 form (34 cycles against 33 for
// the same product), but its accumulators are read and written half as often, and the chip, which lowers its clock under this
// load, draws less power: 18.0 against 20.2 ns per 2 * 65536 operations and SIMD with nothing else running (random codes).  GEMM of
// 8 x 4096 x 4096 -> 4096: 268 us with 32 x 32 x 64, 246 with this; 4 x 8192 x 8192 -> 28672: 2973, 2815.
//
// Operand layout: the 32 codes that one lane feeds to one MFMA (channels 32 f .. 32 f + 31 of a K step of
// 128 channels, f = lane / 16) are a little-endian stream of 6-bit fields = 24 bytes.  A block of 32 rows (columns) is two
// tiles of 16: lane 16 f + i has fragment f of row i of both, 48 bytes, kept as three 16-byte parts.  Per block
// and K step: [3 parts][64 lanes][16 bytes] = 3 KB, so that the 64 lanes of a wave read
// 1 KB of consecutive addresses with one 16-byte LDS read (no bank conflicts, no swizzle; 16-byte reads
// move 1.75x the bytes per clock of 8-byte ones on this chip, and at 8 bytes the fragment reads of a step
// take as long as its MFMAs).  Weights: tile = column / 16 of the block.  Activations (row_off6): the
// rows are dealt to blocks, tiles and lanes so that a lane's results, rows 4 f + v of every tile, are whole blocks of the inverse once
// pairs of lanes have exchanged columns (stamp_epilogue_reg.h).  Per tile and K step, activations: 8 blocks = 24 KB, weights: 4 blocks = 12 KB
// per 128 columns.  The global image equals the LDS image, so a K step is staged by plain asynchronous
// 16-byte copies.
#include <type_traits>

#define STAMP_GEMM6_WAVES 8
#include "stamp_gemm6_kernel.h"
#include "stamp_hi6.h"

namespace {

using namespace stamp_gemm;

// q_lo (tiled [Mpad/256][KT][256 rows][64 bytes], channels in natural order) -> FP6 operand layout.
// One workgroup per (row tile, K step); thread = a fragment of two rows, three 16-byte stores.
// The first nhi blocks convert the 8-bit rows (stamp_hi6.h).
__global__ __launch_bounds__(512) void k_repack6(const uint8_t* __restrict__ q_lo, uint8_t* __restrict__ a6, int nhi, StampHi6Pack hp, int gb) {
  if ((int)blockIdx.x < nhi) {
    hi6_pack(hp, (int)blockIdx.x * 512 + (int)threadIdx.x);
    return;
  }
  repack6_rows(q_lo, a6, blockIdx.x - nhi, threadIdx.x, gb);
}

// The same from rows in STaMP order to rows in the block order of StampRag (rows without a coefficient: zeros).
__global__ __launch_bounds__(512) void k_repack6_rag(const uint8_t* __restrict__ q_lo, uint8_t* __restrict__ a6, StampRag rg, int s,
                                                     int khi, int KT, int M, int nhi, StampHi6Pack hp) {
  if ((int)blockIdx.x < nhi) {
    hi6_pack(hp, (int)blockIdx.x * 512 + (int)threadIdx.x);
    return;
  }
  const int blk = blockIdx.x - nhi, mt = blk / KT, kt = blk - mt * KT;
  const int u = threadIdx.x, m0 = mt * 256 + repack6_row(u, rg.r), R = 1 << rg.r;
  u4 w[2] = {};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + repack6_dist(rg.r) * i, g = m / R, b = g / rg.nb;
    const int slot = m < M ? stamp_rag_slot(rg, g - b * rg.nb, m - g * R) : -1;
    if (slot >= khi) {
      const size_t ms = (size_t)b * s + slot;
      w[i] = *reinterpret_cast<const u4*>(q_lo + (((ms >> 8) * KT + kt) * 256 + (ms & 255)) * 64 + repack6_frag(u) * 16);
    }
  }
  repack6_store(a6 + (size_t)blk * kStageA6 + (u >> 6) * kBlock6 + (u & 63) * 16, w[0], w[1]);
}

// Plan-time weight codes in that layout: per output channel n, code = rne(W_cn * (7 / max)) as in
// the integer engine (round-to-nearest weights, one scale per output channel), stored as E2M3 c / 8.
// One thread per (column, 32-channel fragment).
__global__ __launch_bounds__(256) void k_w_quant6(const float* __restrict__ W, const uint32_t* __restrict__ colmax,
                                                  uint8_t* __restrict__ b6, int d, int N, int Kpad, int Npad, size_t sc,
                                                  size_t sn) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  const int frag = blockIdx.y;  // 32-channel fragment over the whole depth
  if (n >= Npad) return;
  float inv = 0.0f;
  if (n < N) {
    const float a = __uint_as_float(colmax[n]);
    if (a > 0.0f) inv = __fdiv_rn(7.0f, a);
  }
  uint64_t part[3] = {0, 0, 0};
  uint64_t acc = 0;
  int nbits = 0, o = 0;
  for (int i = 0; i < 32; ++i) {
    const int c = frag * 32 + i;
    uint32_t code = 0;
    if (n < N && c < d) {
      float r = rintf(__fmul_rn(W[(size_t)c * sc + (size_t)n * sn], inv));
      r = fminf(fmaxf(r, -7.0f), 7.0f);
      const int q = (int)r;
      code = (uint32_t)(q < 0 ? -q : q) | (q < 0 ? 32u : 0u);
    }
    acc |= (uint64_t)code << nbits;
    nbits += 6;
    if (nbits >= 64) {
      part[o++] = acc;
      nbits -= 64;
      acc = (nbits > 0) ? ((uint64_t)code >> (6 - nbits)) : 0;
    }
  }
  const int KT = Kpad >> 7;
  const int kt = frag >> 2, f = frag & 3;
  // output column n = 64 w + 2 l + ni sits in the 32-column block 2 w + ni at row l: a lane of the GEMM then holds
  // two neighbouring output columns (stamp_epilogue_reg.h)
  const int blk = ((n & 127) >> 6) * 2 + (n & 1), rowb = (n & 63) >> 1;
  uint8_t* dst = b6 + ((size_t)(n >> 7) * KT + kt) * kStageB6 + (size_t)blk * kBlock6 + f * 256 + (rowb & 15) * 16;
  store_frag6(dst, rowb >> 4, part);
}

}  // namespace

size_t stamp_a6_bytes(const stamp_plan* p) { return (size_t)(p->Mpad / 256) * (p->Kpad / 128) * kStageA6; }
size_t stamp_b6_bytes(const stamp_plan* p) { return (size_t)(p->Npad / 128) * (p->Kpad / 128) * kStageB6; }

hipError_t stamp_launch_weight_quant6(const stamp_plan* p, const float* W, const uint32_t* colmax, hipStream_t st) {
  const int d = p->geom.d, N = p->geom.N;
  const size_t sc = p->desc.w_is_out_by_in ? 1 : (size_t)N;
  const size_t sn = p->desc.w_is_out_by_in ? (size_t)d : 1;
  hipLaunchKernelGGL(k_w_quant6, dim3((p->Npad + 255) / 256, p->Kpad / 32), dim3(256), 0, st, W, colmax, p->qW6_dev, d, N,
                     p->Kpad, p->Npad, sc, sn);
  return hipGetLastError();
}

hipError_t stamp_launch_repack6(const stamp_plan* p, const uint8_t* q_lo, uint8_t* a6, hipStream_t st, const StampHi6Pack* hi) {
  const int nlo = q_lo != nullptr ? (p->Mpad / 256) * (p->Kpad / 128) : 0;
  const StampHi6Pack hp = hi != nullptr ? *hi : StampHi6Pack{};
  const int nhi = (hp.threads + 511) / 512;
  if (nlo + nhi > 0) hipLaunchKernelGGL(k_repack6, dim3(nlo + nhi), dim3(512), 0, st, q_lo, a6, nhi, hp, stamp_row_group_bit(p));
  return hipGetLastError();
}

size_t stamp_rag_a6_bytes(const stamp_plan* p) {
  const size_t M = (size_t)p->geom.B * p->rag.nb << p->rag.r;
  return ((M + 255) / 256) * (p->Kpad / 128) * kStageA6;
}

hipError_t stamp_launch_repack6_rag(const stamp_plan* p, const uint8_t* q_lo, uint8_t* a6, hipStream_t st, const StampHi6Pack* hi) {
  const int M = (p->geom.B * p->rag.nb) << p->rag.r, KT = p->Kpad / 128, nlo = ((M + 255) / 256) * KT;
  const StampHi6Pack hp = hi != nullptr ? *hi : StampHi6Pack{};
  const int nhi = (hp.threads + 511) / 512;
  hipLaunchKernelGGL(k_repack6_rag, dim3(nlo + nhi), dim3(512), 0, st, q_lo, a6, p->rag, p->geom.s, p->geom.khi, KT, M, nhi, hp);
  return hipGetLastError();
}

// 128 x 256 tiles where the rounds they need (tiles over CUs, rounded up), at two thirds of a round of 256 x 256 tiles each,
// take less time.  Depth 4096, 1-D blocks of 32, 2048 rows, microseconds, 256 x 256 against 128 x 256: 128 tiles of 256 x 256
// 28.3, 23.0; 344 (2 rounds against 3) 58.1, 57.4; depth 11008, 128 tiles: 64.4, 47; at full rounds (256 tiles) 35.8 against
// twice 23.  (Measured while both multiplied with 32 x 32 x 64 MFMAs.)  With 16 x 16 x 128 ones and 8-bit rows in the tiles, whole
// layers, us, 256 x 256 (or pairs of 128 x 256, if stamp_gemm6_pairs takes them) against 128 x 256: half a round 43 against 33 (2048 x 4096 ->
// 4096, 3 levels), 57 against 48 (8192 x 4096 -> 1024); 0.56 to 0.6 rounds 27.2, 29.2 (4096 x 1152 -> 2304); two rounds against three, 2048
// -> 8448 .. 11008, 3 levels: depth 1152 38.4, 36.5, 4096 78.3, 74.3, 8192 137.4, 138.5; without transform 1152 37.4, 41.7, 4096 76.6,
// 77.3; full depth 4096 93.0, 92.2, 8192 156, 166.  The line stands where it was.
bool stamp_gemm6_half_tiles(int M, int Npad) {
  const int cus = stamp_device_cus(), nt = Npad / BN6;
  const int r8 = ((M + 255) / 256 * nt + cus - 1) / cus, r4 = ((M + 127) / 128 * nt + cus - 1) / cus;
  return 100 * r8 > 68 * r4;
}

// Two workgroups of 128 x 256 tiles per CU against one of 256 x 256.  Layers of 8192 rows, us, by K steps and rounds (256 x 256 tiles over CUs);
// last where the last round is up to half full, then fuller, then full.  Fused, 3 levels: 5 steps: 1.1 to 1.5 rounds 36.0, 32.5, 2.25 49.0,
// 44.3, 2.5 49.2, 45.0; 1.75 37.2, 35.6; 2 42.3, 36.9, 3 52.2, 52.6, 4 70.7, 64.7.  9: 1.1 46.1, 41.8, 1.5 46.0, 41.9, 2.25 62.7, 56.7; 1.75 46.6, 45.1; 2
// 53.4, 47.9, 3 67.2, 67.1, 4 89.5, 81.3.  16: 1.1 58.0, 54.3, 1.5 58.4, 56.3, 2.25 80.5, 76.0; 1.75 62.0, 61.6; 2 67.3, 63.6, 3 88.0, 88.5, 4 115.3, 112.0.
// 32: 1.1 91.0, 90.0, 1.5 96.2, 92.3, 2.25 129.1, 126.8; 1.75 96.4, 99.2; 2 103.6, 103.8, 3 144.3, 146.9.  Blocks of any length and token grids the same but
// for 1.6 rounds of a grid with rows that are no whole lines, 704 -> 3080: 46.6, 49.2.  Depth 8192, 56 rounds: 2743, 3567 the GEMM alone.
// Without transform: 5: 1.1 33.8, 31.6, 2.25 46.9, 44.2; 2 37.8, 35.4, 3 48.8, 48.4, 4 68.3, 62.1.  9: 1.1 41.9, 39.1, 2.25 58.2, 54.4; 1.75 43.7, 43.6; 2
// 46.9, 44.5, 3 61.4, 61.0.  16: 1.1 53.6, 51.8, 2.25 76.9, 74.3; 1.75 56.7, 58.0; 2 59.6, 59.9, 3 82.9, 85.6.  32: 1.1 87.4, 88.8, 2.25 123.8, 125.8.
// fp32 rows (the whole WHT layer): 5: 1.1 103.1, 100.8, 1.5 125.3, 123.3, 2.25 179.1, 180.6; 2 161, 153.  9: 1.1 112.7, 111.4, 2.25 172.2, 174.3; 2 146.1,
// 145.8, 3 212.7, 214.3.  16: 1.1 137.8, 135.9, 1.5 144.8, 144.1, 2.25 207.8, 211.1; 2 171.8, 174.1.  32: 1.1 200.8, 202.0, 2 240, 249.
// Hence: last rounds up to half full, which pairs halve, and shallow layers' full ones, whose stores come all at once in 256 x 256 tiles.
bool stamp_gemm6_pairs(int M, int Npad, int Kpad, int mode) {
  const int cus = stamp_device_cus(), kt = Kpad / BK;
  const int64_t tiles = (int64_t)((M + 127) / 128) * (Npad / BN6), rem = tiles % (2 * cus), two = 4 * (int64_t)cus;  // two: of full rounds
  if (mode == 0 || tiles <= 2 * cus || rem > cus) return false;
  if (kt <= 9) return mode != 1 || tiles <= two;
  if (mode == 1) return false;
  if (rem == 0) return mode == 2 && kt <= 24 && tiles == two;
  return kt <= (mode == 2 ? 32 : 24);
}

namespace {
hipError_t gemm6(const GemmArgs& a, int mode, hipStream_t st) {
  if (a.ht.on) return mode == 2 ? stamp_gemm6_half_hi(a, st) : hipErrorInvalidValue;
  if (mode != 0 && stamp_gemm6_half_tiles(a.M, a.Npad)) return stamp_gemm6_half(a, mode, st);
  return stamp_gemm6_pairs(a.M, a.Npad, a.Kpad, mode) ? stamp_gemm6_pair(a, mode, st) : gemm6_run(a, mode, st);
}
}  // namespace

hipError_t stamp_launch_gemm_lo6_rag(const stamp_plan* p, const uint8_t* a6, const float* scales, void* Y, const float* P, hipStream_t st,
                                     const StampHiOut* hi) {
  GemmArgs a = stamp_gemm_args(p, scales, Y);
  a.A = a6;
  a.Bq = p->qW6_dev;
  a.g = p->bgeom;
  a.rag = p->rag;
  a.gb = p->rag.r;
  a.M = a.g.B * a.g.k * a.g.R;
  a.P = P;
  if (hi != nullptr) {
    a.H = hi->p;
    a.ht = hi->ht;
  }
  return gemm6(a, 2, st);
}

hipError_t stamp_launch_gemm_lo6(const stamp_plan* p, const uint8_t* a6, const float* scales, int mode, void* out,
                                 const float* P, hipStream_t st, int own_top, const StampHiOut* hi) {
  GemmArgs a = stamp_gemm_args(p, scales, out);
  a.A = a6;
  a.Bq = p->qW6_dev;
  a.M = p->geom.B * p->geom.s;
  a.P = P;
  a.own_top = (mode == 2) ? own_top : 0;
  if (hi != nullptr) {
    a.H = hi->p;
    a.ht = hi->ht;
  }
  return gemm6(a, mode, st);
}
