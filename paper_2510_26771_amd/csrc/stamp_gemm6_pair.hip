// The FP6 GEMM on 128 x 256 tiles, two workgroups per CU.
#define STAMP_GEMM6_WAVES 4
#define STAMP_GEMM6_PAIR
#include "stamp_gemm6_kernel.h"

hipError_t stamp_gemm6_pair(const stamp_gemm::GemmArgs& a, int mode, hipStream_t st) { return gemm6_run(a, mode, st); }
