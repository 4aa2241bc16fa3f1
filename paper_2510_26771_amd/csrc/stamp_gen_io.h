// Shared by the kernels of the general path: elements in and out, complex numbers in fp64.
#ifndef STAMP_GEN_IO_H_
#define STAMP_GEN_IO_H_

#include "stamp_internal.h"

namespace {

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// One element of the input of a transform pass: X itself (bf16 or fp32) or an fp32 work buffer.
__device__ __forceinline__ float gen_load(const void* in, int kind, size_t idx) {
  return kind == 2 ? __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(in)[idx] << 16) : reinterpret_cast<const float*>(in)[idx];
}
// n elements, `step` apart.  One branch on the type for all of them: a branch per element would make every load wait for
// the one before it (s = 2048, 4096 channels, 32 rows per thread: WHT 41 -> 25 us).
template <int n>
__device__ __forceinline__ void gen_load_rows(const void* in, int kind, size_t idx, size_t step, float (&v)[n]) {
  if (kind == 2) {
    uint32_t w[n];
#pragma unroll
    for (int j = 0; j < n; ++j) w[j] = reinterpret_cast<const uint16_t*>(in)[idx + j * step];
#pragma unroll
    for (int j = 0; j < n; ++j) v[j] = __uint_as_float(w[j] << 16);
  } else {
#pragma unroll
    for (int j = 0; j < n; ++j) v[j] = reinterpret_cast<const float*>(in)[idx + j * step];
  }
}
__device__ __forceinline__ void gen_store_y(void* Y, int y_bf16, size_t idx, float v) {
  if (y_bf16) reinterpret_cast<uint16_t*>(Y)[idx] = f32_to_bf16_rne(v);
  else reinterpret_cast<float*>(Y)[idx] = v;
}

struct cd {
  double re, im;
};
__device__ __forceinline__ cd c_add(cd a, cd b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cd c_sub(cd a, cd b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cd c_mul(cd a, cd b) {
  return {__builtin_fma(a.re, b.re, -(a.im * b.im)), __builtin_fma(a.re, b.im, a.im * b.re)};
}
__device__ __forceinline__ cd c_conj(cd a) { return {a.re, -a.im}; }
// An infinity enters as a number far beyond the range of fp32, so that every coefficient it is part of leaves as an infinity
// of its sign, as in the sum that defines it; an infinity itself would meet 0 * inf in the first product with a factor and
// leave NaNs, which the row maxima of the quantizer pass over.  One test for all of a thread's values.
template <int n>
__device__ __forceinline__ void dct_in(const float (&x)[n], double (&v)[n]) {
  float m = 0.0f;
#pragma unroll
  for (int j = 0; j < n; ++j) {
    m = fmaxf(m, fabsf(x[j]));
    v[j] = (double)x[j];
  }
  if (__builtin_isinf(m)) {
#pragma unroll
    for (int j = 0; j < n; ++j)
      if (__builtin_isinf(x[j])) v[j] = __builtin_copysign(1e300, v[j]);
  }
}

}  // namespace

#endif  // STAMP_GEN_IO_H_
