// The FP6 GEMM on 128 x 256 tiles that takes the 8-bit rows along.
#define STAMP_GEMM6_WAVES 4
#define STAMP_GEMM6_HI
#include "stamp_gemm6_kernel.h"

hipError_t stamp_gemm6_half_hi(const stamp_gemm::GemmArgs& a, hipStream_t st) { return gemm6_run(a, 2, st); }
