// Bottom kernels of 1-D blocks of 16 tokens (a file per block length: they compile side by side).
#include "stamp_bottom_kernel.h"

hipError_t stamp_bottom1d_4(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split,
                            hipStream_t st) {
  const SplitArgs& sp = *static_cast<const SplitArgs*>(split);
  const StampGeom& g = p->geom;
  if (g.asym) return g.x_bf16 ? launch_bottom1d<4, true, true>(p, X, q_lo, scales, abot, nthreads, sp, st)
                              : launch_bottom1d<4, false, true>(p, X, q_lo, scales, abot, nthreads, sp, st);
  return g.x_bf16 ? launch_bottom1d<4, true, false>(p, X, q_lo, scales, abot, nthreads, sp, st)
                  : launch_bottom1d<4, false, false>(p, X, q_lo, scales, abot, nthreads, sp, st);
}

hipError_t stamp_bottom1d_rag_4(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const StampHiOut& hi6, hipStream_t st) {
  return launch_rag_t<4>(p, X, q_hi, q_lo, scales, hi6, st);
}
