// FP6 (E2M3) operand format of the GEMMs on the FP6 matrix pipeline: constants of the layout (described in
// stamp_gemm6.hip) and the conversion of 4-bit codes.
#ifndef STAMP_FP6_H_
#define STAMP_FP6_H_

#include "stamp_gemm_common.h"

namespace stamp_gemm {

typedef int v6i __attribute__((ext_vector_type(6)));
typedef uint32_t u6 __attribute__((ext_vector_type(6)));
// the FP6 operand of the MFMA builtin is declared as 8 registers, of which the instruction reads 6
__device__ __forceinline__ v8i widen(v6i x) { return __builtin_shufflevector(x, x, 0, 1, 2, 3, 4, 5, -1, -1); }

constexpr int kPart = 2 * 32 * 16;            // bytes of one part of a 32-row block: 1 KB
constexpr int kBlock6 = 3 * kPart;            // a 32-row block of one K step: 3 KB
constexpr int kStageB6 = 4 * kBlock6;         // 128 columns: 12 KB
constexpr int kStageA6 = 2 * kStageB6;        // 24 KB

// Activation rows.  Bit gb of a row (2 .. 6; bit 7: which half of a 256-row tile) is the group of 32 lanes that its results come out
// in, the other six of bits 0 .. 6 are its place there, L: bits 0 and 1 the result register, 2 the lanes of the group, 3 which of a lane's
// two operands (tiles of 16 rows), 4 and 5 the block.  gb = log2 of the rows that the epilogue keeps together in a lane, at least 2: the
// two groups hold neighbouring blocks (plain rows: neighbouring four rows), and both have work in a tile with few rows.  With bit 6 for
// all plans one of them had none where a tile has up to 64: 64 x 256 -> 128 18.7 us, 18.2 with this; 64 x 512 -> 4096 19.9, 19.6; 40 x 1024 ->
// 4096 without transform 17.1, 16.5; 77 x 2048 -> 1024 21.2, 20.4.  Blocks of 64: place_of_64.
STAMP_HD uint32_t row_rest6(uint32_t r, int gb) {
  const uint32_t L = ((r & 127) >> (gb + 1) << gb) | (r & ((1u << gb) - 1));
  return gb == 6 ? place_of_64(L) : L;
}
STAMP_HD bool row_half6(uint32_t r, int gb) { return (row_rest6(r, gb) >> 3) & 1; }
// row of a 256-row tile -> byte of its lane in channels 0 .. 31 of K step 0
STAMP_HD uint32_t row_off6(uint32_t r, int gb) {
  const uint32_t L = row_rest6(r, gb);
  return (((r >> 5) & 4) + (L >> 4)) * (uint32_t)kBlock6 + (((r >> gb) & 1) * 8 + (L & 7)) * 16;
}
// row of a block of 8-bit rows, which stand by themselves: bits 0, 1, 3 and 4 choose the lane, bit 2 the operand
STAMP_HD uint32_t row_lane6(uint32_t r) { return (((r >> 1) & 12) + (r & 3)) * 16; }
STAMP_HD bool hi_half6(uint32_t r) { return (r >> 2) & 1; }
// byte offset of the 32 channels from c on; K steps are kt_bytes apart
STAMP_HD uint32_t chan_off6(uint32_t c, uint32_t kt_bytes) { return (c >> 7) * kt_bytes + ((c >> 5) & 3) * 256; }

typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u6v __attribute__((ext_vector_type(6)));
// 24 bytes of a fragment -> their places; dst = its lane's place in part 0, half = row_half6 of the row (8-bit rows: hi_half6)
__device__ __forceinline__ void store24(uint8_t* dst, u6v w, bool half) {
  const u4 a = {half ? w[2] : w[0], half ? w[3] : w[1], half ? w[4] : w[2], half ? w[5] : w[3]};
  const u2 b = {half ? w[0] : w[4], half ? w[1] : w[5]};
  *reinterpret_cast<u4*>(dst + (half ? 2 * kPart : 0)) = a;
  *reinterpret_cast<u2*>(dst + kPart + (half ? 8 : 0)) = b;
}
// channels 2 i in ev[i], 2 i + 1 in od[i]: integers of magnitude up to 8 (or values that round to such)
// (An asm statement, so that the result has registers of its own: the instruction writes before it has read everything, and the builtin's
// result was placed across its operands: results from v4 on, operands from v2 on, came out wrong.)
__device__ __forceinline__ u6v to_e2m3(f16v ev, f16v od) {
  u6v r;
  asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3" : "=&v"(r) : "v"(ev), "v"(od), "s"(8.0f));
  return r;
}
// codes 16 h + l of magnitude up to 128 -> the fragments of h and l, l in [-8, 7]
__device__ __forceinline__ void split_hi(f16v ev, f16v od, u6v& h, u6v& l) {
  f16v hv[2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) hv[p][i] = floorf(__builtin_fmaf(p ? od[i] : ev[i], 0.0625f, 0.5f));
  h = to_e2m3(hv[0], hv[1]);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    ev[i] = __builtin_fmaf(-16.0f, hv[0][i], ev[i]);
    od[i] = __builtin_fmaf(-16.0f, hv[1][i], od[i]);
  }
  l = to_e2m3(ev, od);
}

// the same by words, for fragments put together bit by bit
__device__ __forceinline__ void store_frag6(uint8_t* dst, bool half, const uint64_t (&part)[3]) {
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const int off = (half ? 24 : 0) + w * 8;
    *reinterpret_cast<uint64_t*>(dst + (off >> 4) * kPart + (off & 15)) = part[w];
  }
}

// eight two's-complement nibbles -> eight sign-magnitude 6-bit fields
__device__ __forceinline__ void nib8_to_48(uint32_t w, uint32_t& w0, uint32_t& w1) {
  const uint32_t s = w & 0x88888888u, sg = s >> 3;
  // |c|: complement the negative nibbles and add 1 (no carry leaves a nibble: ~c + 1 <= 8).  |c| = 8
  // (the stored form of the asymmetric code 0) sets the low exponent bit: the E2M3 number 1.0 = 8 / 8.
  const uint32_t mag = (w ^ ((s << 1) - sg)) + sg;
  auto spread = [](uint32_t x) {  // four nibbles to bits 0, 6, 12, 18
    const uint32_t t = (x & 0x00FFu) | ((x & 0xFF00u) << 4);
    return (t & 0x00F00Fu) | ((t & 0x0F00F0u) << 2);
  };
  const uint32_t lo = spread(mag & 0xFFFFu) | (spread(sg & 0xFFFFu) << 5), hi = spread(mag >> 16) | (spread(sg >> 16) << 5);
  w0 = lo | (hi << 24);
  w1 = hi >> 8;
}

// 32 codes (one 16-byte chunk of packed nibbles, low nibble = even channel) -> 24 bytes
__device__ __forceinline__ void chunk_to_e2m3(u4 w, uint64_t (&part)[3]) {
  uint32_t lo[4], hi[4];
  nib8_to_48(w.x, lo[0], hi[0]);
  nib8_to_48(w.y, lo[1], hi[1]);
  nib8_to_48(w.z, lo[2], hi[2]);
  nib8_to_48(w.w, lo[3], hi[3]);
  part[0] = lo[0] | ((uint64_t)(hi[0] | (lo[1] << 16)) << 32);
  part[1] = ((lo[1] >> 16) | (hi[1] << 16)) | ((uint64_t)lo[2] << 32);
  part[2] = (hi[2] | (lo[3] << 16)) | ((uint64_t)((lo[3] >> 16) | (hi[3] << 16)) << 32);
}

}  // namespace stamp_gemm

#endif  // STAMP_FP6_H_
