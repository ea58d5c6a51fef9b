// The inverse of a 16 x 16 float64 block inside one wave.
#pragma once
#include <hip/hip_runtime.h>

namespace osscar {

typedef double swd4 __attribute__((ext_vector_type(4)));
// lane k of each row of 16 lanes, to all 16 of them
template <int K>
__device__ __forceinline__ double row16_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + K, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + K, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
// Pivots K.. of the Gauss-Jordan inverse of a 16 x 16 block that one wave holds like a result of v_mfma_f64_16x16x4_f64:
// x[r] = element (4 r + lane / 16, lane % 16).  The pivot row crosses the rows of lanes by one ds_bpermute (two dwords),
// the pivot column and the pivot itself by DPP broadcasts.
template <int K>
__device__ __forceinline__ void inv16_steps(swd4& x, int lane, int n, bool& flag) {
  if constexpr (K < 16) {
    if (K >= n) return;                    // uniform: rows and columns from n on behave as an identity block
    const int from = (((K & 3) << 4) | (lane & 15)) << 2;
    const double mine = x[K >> 2];
    const double row = __hiloint2double(__builtin_amdgcn_ds_bpermute(from, __double2hiint(mine)),
                                        __builtin_amdgcn_ds_bpermute(from, __double2loint(mine)));
    // the pivot goes by v_readlane, ahead of the row; its reciprocal is a division, rounded correctly and 0 for an infinite pivot
    // (v_rcp_f64 and two Newton steps are not, and give NaN there; the inverse of 128 rows takes 37 us either way, and a layer of
    // 256 groups of nine between the same 8.5 ms and 0.2 ms more)
    double piv = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(mine), ((K & 3) << 4) | K),
                                  __builtin_amdgcn_readlane(__double2loint(mine), ((K & 3) << 4) | K));
    if (!(piv > 0.0)) { flag = true; piv = 1.0; }
    const double d = 1.0 / piv;
    const double rs = row * d;
    const bool pcol = (lane & 15) == K, prow = (lane >> 4) == (K & 3);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const double c = row16_bcast<K>(x[r]);
      const double v = x[r] - c * rs;
      x[r] = pcol ? -c * d : v;
    }
    if (prow) x[K >> 2] = pcol ? d : rs;
    inv16_steps<K + 1>(x, lane, n, flag);
  }
}

}  // namespace osscar
