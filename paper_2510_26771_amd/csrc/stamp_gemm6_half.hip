// The FP6 GEMM on 128 x 256 tiles (4 waves): a file of its own, so that the two sets of kernels compile side by side.
#define STAMP_GEMM6_WAVES 4
#include "stamp_gemm6_kernel.h"

hipError_t stamp_gemm6_half(const stamp_gemm::GemmArgs& a, int mode, hipStream_t st) { return gemm6_run(a, mode, st); }
