// Device code that the files of the delayed-update search share.
#pragma once
#include "internal.h"

namespace osscar {

// pending pivots including those of the iteration that ran last (for kernels outside an iteration)
__device__ __forceinline__ int tau_all(const SearchCtrl* c) { return c->tau + c->tau_inc; }
// the pending set is empty from here on; by one workgroup of nt threads
__device__ __forceinline__ void empty_pending(const LazyPtrs& L, SearchCtrl* ctrl, int nt) {
  const int tau = tau_all(ctrl);
  for (int s = threadIdx.x; s < tau; s += nt) L.pos[L.Tidx[s]] = -1;
  __syncthreads();
  if (threadIdx.x == 0) { ctrl->tau = 0; ctrl->tau_inc = 0; ctrl->pause = 0; ctrl->spare = L.spare0; }
}
// the score of a row from its squared norm and diagonal element
__device__ __forceinline__ double fresh_score(int h, const int32_t* __restrict__ kept, const double* __restrict__ gram, const double* __restrict__ dblk,
                                              double* __restrict__ score, SearchCtrl* ctrl) {
  double a = (kept[h] ? -1.0 : 1.0) * dblk[h];
  if (!(a > 0.0)) { ctrl->notpd = 1; a = 1.0; }
  return score[h] = gram[h] / a;
}

}  // namespace osscar
