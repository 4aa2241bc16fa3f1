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

// eight two's-complement nibbles -> eight sign-magnitude 6-bit fields (48 bits)
__device__ __forceinline__ uint64_t nib8_to_e2m3(uint32_t w) {
  const uint32_t s = w & 0x88888888u;  // sign bit of every nibble
  const uint32_t sg = s >> 3;          // 1 in every negative nibble
  // |c|: complement the negative nibbles and add 1 (no carry leaves a nibble: ~c + 1 <= 8).  |c| = 8
  // (the stored form of the asymmetric code 0) sets the low exponent bit: the E2M3 number 1.0 = 8 / 8.
  const uint32_t mag = (w ^ (sg * 15u)) + sg;
  uint64_t out = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t c = ((mag >> (4 * j)) & 15u) | (((s >> (4 * j + 3)) & 1u) << 5);
    out |= (uint64_t)c << (6 * j);
  }
  return out;
}

// 32 codes (one 16-byte chunk of packed nibbles, low nibble = even channel) -> 24 bytes
__device__ __forceinline__ void chunk_to_e2m3(u4 w, uint64_t (&part)[3]) {
  const uint64_t a = nib8_to_e2m3(w.x), b = nib8_to_e2m3(w.y), c = nib8_to_e2m3(w.z), d = nib8_to_e2m3(w.w);
  part[0] = a | (b << 48);
  part[1] = (b >> 16) | (c << 32);
  part[2] = (c >> 32) | (d << 16);
}

// 32 signed values of magnitude at most 8 -> 24 bytes of E2M3 numbers value / 8
__device__ __forceinline__ void values_to_e2m3(const int (&v)[32], uint64_t (&part)[3]) {
#pragma unroll
  for (int w = 0; w < 3; ++w) part[w] = 0;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const uint64_t f = (uint64_t)((uint32_t)abs(v[i]) | ((uint32_t)(v[i] >> 31) & 32u));
    const int bit = 6 * i, w = bit >> 6, sh = bit & 63;
    part[w] |= f << sh;
    if (sh > 58) part[w + 1] |= f >> (64 - sh);
  }
}

}  // namespace stamp_gemm

#endif  // STAMP_FP6_H_
