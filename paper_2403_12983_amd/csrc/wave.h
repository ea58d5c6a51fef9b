// Reductions and small helpers of the search kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace osscar {

__device__ __forceinline__ float nsym1(const float* __restrict__ N, int64_t ld, int i, int t) {
  return (i >= t) ? N[(int64_t)i * ld + t] : N[(int64_t)t * ld + i];
}
// Sum over the 64 lanes of a wave by data-parallel-primitive moves (no trip through the LDS crossbar, which costs a
// shuffle about 40 ns here and made the reductions the longest part of the small kernels): pairs and quads by quad
// permutations, the four quads of a row of 16 by row rotations, then row 0 -> 1 and 2 -> 3 (row_bcast:15) and
// rows 0-1 -> 3 (row_bcast:31); lane 63 holds the total, which every lane receives.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_get(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROW_MASK, 0xf, false);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROW_MASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_get_or(double v, double dflt) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_update_dpp(__double2loint(dflt), lo, CTRL, ROW_MASK, 0xf, false);
  hi = __builtin_amdgcn_update_dpp(__double2hiint(dflt), hi, CTRL, ROW_MASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_get_or(int v, int dflt) { return __builtin_amdgcn_update_dpp(dflt, v, CTRL, ROW_MASK, 0xf, false); }
__device__ __forceinline__ double wsum(double v) {
  v += dpp_get<0xb1, 0xf>(v);        // quad_perm [1, 0, 3, 2]
  v += dpp_get<0x4e, 0xf>(v);        // quad_perm [2, 3, 0, 1]
  v += dpp_get<0x124, 0xf>(v);       // row_ror:4
  v += dpp_get<0x128, 0xf>(v);       // row_ror:8
  v += dpp_get<0x142, 0xa>(v);       // row_bcast:15 into rows 1 and 3 (other rows add zero)
  v += dpp_get<0x143, 0xc>(v);       // row_bcast:31 into rows 2 and 3
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63), hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}
// Sum over each group of eight consecutive lanes (every lane of the group receives it): pairs and quads by quad
// permutations, the two quads of a half row by row_half_mirror (lane i of the half row reads lane 7 - i, which by then
// holds the other quad's sum).
__device__ __forceinline__ double sum8(double v) {
  v += dpp_get<0xb1, 0xf>(v);
  v += dpp_get<0x4e, 0xf>(v);
  v += dpp_get<0x141, 0xf>(v);
  return v;
}

// (value, index): the smaller value, the lower index on ties, index -1 = none; six data-parallel steps leave the best of the
// wave in lane 63
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void dpp_min_step(double& v, int& i) {
  const double ov = dpp_get_or<CTRL, ROW_MASK>(v, INFINITY);
  const int oi = dpp_get_or<CTRL, ROW_MASK>(i, -1);
  const bool t = (oi >= 0) & ((i < 0) | (ov < v) | ((ov == v) & (oi < i)));      // (no branches)
  v = t ? ov : v; i = t ? oi : i;
}
__device__ __forceinline__ void wave_min(double& v, int& i) {
  dpp_min_step<0xb1, 0xf>(v, i); dpp_min_step<0x4e, 0xf>(v, i); dpp_min_step<0x124, 0xf>(v, i);
  dpp_min_step<0x128, 0xf>(v, i); dpp_min_step<0x142, 0xa>(v, i); dpp_min_step<0x143, 0xc>(v, i);
}
__device__ __forceinline__ double wave_min(double v) {
  v = fmin(v, dpp_get_or<0xb1, 0xf>(v, INFINITY)); v = fmin(v, dpp_get_or<0x4e, 0xf>(v, INFINITY));
  v = fmin(v, dpp_get_or<0x124, 0xf>(v, INFINITY)); v = fmin(v, dpp_get_or<0x128, 0xf>(v, INFINITY));
  v = fmin(v, dpp_get_or<0x142, 0xa>(v, INFINITY)); v = fmin(v, dpp_get_or<0x143, 0xc>(v, INFINITY));
  return v;
}

}  // namespace osscar
