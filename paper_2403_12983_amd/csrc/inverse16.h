// The inverse of a 16 x 16 float64 block inside one wave.
#pragma once
#include <hip/hip_runtime.h>

namespace osscar {

typedef double swd4 __attribute__((ext_vector_type(4)));
// Pivots 2 S, 2 S + 1, .. of the symmetric sweep of a 16 x 16 block that one wave holds like a result of v_mfma_f64_16x16x4_f64: x[r] = element
// (4 r + lane / 16, lane % 16).  The two pivot rows lie in one register as that instruction's operand has them, and by symmetry the pivot columns
// are the same numbers, so a step is two matrix instructions: T = D R (D: the inverse of the 2 x 2 pivot block, R: the pivot rows) and
// X - T^T R; the pivot columns, zeroed before, receive T through columns of -1 in R's place.
// Bound by the chain of steps: 2 x 2 block by v_readlane, two divisions, two matrix instructions.  Eight steps; pivot by
// pivot, a row through ds_bpermute each, the inverse of 100 rows took 5 us (a tenth) longer.
template <int S>
__device__ __forceinline__ void sweep16_pairs(swd4& x, int lane, int n, bool& flag) {
  if constexpr (S < 8) {
    if (2 * S >= n) return;                // uniform: rows and columns from n on behave as an identity block
    constexpr int P = 2 * S, R0 = S >> 1, G0 = 2 * (S & 1);
    const int lr = lane >> 4, lc = lane & 15;
    const double own = x[R0];
    auto at = [&](int l) { return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(own), l), __builtin_amdgcn_readlane(__double2loint(own), l)); };
    // the pivots one after the other, each reciprocal a division: rounded correctly, and 0 for an infinite pivot
    double a = at(16 * G0 + P);
    const double b = at(16 * G0 + P + 1), c = at(16 * (G0 + 1) + P + 1);
    if (!(a > 0.0)) { flag = true; a = 1.0; }
    const double d = 1.0 / a, u = b * d;
    double e = c - b * u;
    if (!(e > 0.0)) { flag = true; e = 1.0; }
    const double d22 = 1.0 / e, d12 = -u * d22, d11 = d - u * d12;
    const bool row = (lr >> 1) == (S & 1), col = lc == P || lc == P + 1, same = lc - P == lr - G0;
    const double dk = lr == G0 ? d11 : d22;
    const swd4 zero = {0.0, 0.0, 0.0, 0.0};
    const swd4 t = __builtin_amdgcn_mfma_f64_16x16x4f64(row && (lc >> 1) == (S & 1) ? (lc == lr ? dk : d12) : 0.0, own, zero, 0, 0, 0);
    const double tt = t[0];                // T in the lanes of the pivot rows, zero elsewhere
    swd4 y;
#pragma unroll
    for (int r = 0; r < 4; r++) y[r] = col ? 0.0 : x[r];
    y = __builtin_amdgcn_mfma_f64_16x16x4f64(-tt, col ? (same ? -1.0 : 0.0) : own, y, 0, 0, 0);
    if (row) y[R0] = col ? (same ? -dk : -d12) : tt;
    x = y;
    sweep16_pairs<S + 1>(x, lane, n, flag);
  }
}
// the inverse of the leading n x n part of such a block (symmetric positive definite; a pivot block that is not sets flag)
__device__ __forceinline__ void inv16(swd4& x, int lane, int n, bool& flag) {
  sweep16_pairs<0>(x, lane, n, flag);
#pragma unroll
  for (int r = 0; r < 4; r++) x[r] = -x[r];
}

}  // namespace osscar
