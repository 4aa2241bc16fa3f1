// Bottom kernels of 1-D blocks of 128 tokens (a file per block length: they compile side by side).
#include "stamp_bottom_kernel.h"

hipError_t stamp_bottom1d_7(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads, const void* split,
                            hipStream_t st) {
  const SplitArgs& sp = *static_cast<const SplitArgs*>(split);
  const StampGeom& g = p->geom;
  if (g.asym) return g.x_bf16 ? launch_bottom1d<7, true, true>(p, X, q_lo, scales, abot, nthreads, sp, st)
                              : launch_bottom1d<7, false, true>(p, X, q_lo, scales, abot, nthreads, sp, st);
  return g.x_bf16 ? launch_bottom1d<7, true, false>(p, X, q_lo, scales, abot, nthreads, sp, st)
                  : launch_bottom1d<7, false, false>(p, X, q_lo, scales, abot, nthreads, sp, st);
}
