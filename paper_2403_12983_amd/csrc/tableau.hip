// The swept tableau and the kernels of the local search (Section 4.2; Proposition 4.1, Cases 1-3).
//
// State.  For the kept set K the library holds the symmetric d1 x d1 matrix
//        N = [ -P   V ]      P = (H_KK)^-1,  V = P H_{K,Kc},  S = H_cc - H_cK P H_Kc
//            [ V^T  S ]
// in the ORIGINAL row order (row i belongs to group i / q, kept or not), lower triangle only, and
//        Z = [ B ; R ]       B = P G_K (optimal kept weights),  R = G_Kc - H_cK B
// as d1 x m.  N is H with the "sweep operator" applied to the pivots in K, and Z is G carried along.
// In this form Proposition 4.1's Case 2 (a group enters) is a forward sweep on that group's q x q
// pivot block and Case 1 (a group leaves) is the reverse sweep; both are the same rank-q update
//        N_il -= N_it D N_tl,   Z_i -= N_it D Z_t        (D = N_tt^-1, i, l outside the pivot)
// and differ only in the sign given to the pivot rows (+D N_tl entering, -D N_tl leaving; N_tt' = -D).
// The change of the objective is -Tr(Z_t^T D Z_t) in both cases, and the impact score of eq. (impact)
// of ANY group h is Tr(Z_h^T |N_hh|^-1 Z_h): removal cost if h is kept, addition gain otherwise.
// A swap (Case 3) is the reverse sweep on g followed by the forward sweep on j; the two are fused into
// one rank-2q pass over N and Z, with the second pivot's panel corrected for the first sweep beforehand.
#include "internal.h"
#include "inverse16.h"
#include <algorithm>

namespace osscar {

// ------------------------------------------------------------------------------------------------
// small dense helpers (float64, one workgroup, matrices in global or shared memory)
// ------------------------------------------------------------------------------------------------
// In-place inverse of the n x n matrix A (leading dimension n, n <= 16 T, shared or global memory) by Gauss-Jordan without
// pivoting; valid for definite matrices of either sign.  want_sign = +1 / -1: every pivot must have that sign, else
// *bad = 1.  Called by all 256 threads of a workgroup: thread (ti, tj) of a 16 x 16 grid keeps the T x T block with rows
// ti*T.. and columns tj*T.. in registers (rows and columns past n behave as an identity block); every step broadcasts the
// pivot row and column through buf (64 T doubles of shared memory, two halves used in turn: one barrier per step).
template <int T>
__device__ void small_inverse(double* A, int n, int want_sign, int32_t* bad, double* buf) {
  const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
  double r[T][T];
  __syncthreads();
#pragma unroll
  for (int a = 0; a < T; a++)
#pragma unroll
    for (int b = 0; b < T; b++) {
      const int i = ti * T + a, j = tj * T + b;
      r[a][b] = (i < n && j < n) ? A[i * n + j] : (i == j ? 1.0 : 0.0);
    }
  bool flag = false;
  for (int k0 = 0; k0 < n; k0 += T) {
#pragma unroll
    for (int kk = 0; kk < T; kk++) {
      const int k = k0 + kk;
      if (k < n) {                                   // uniform over the workgroup
        double* rowb = buf + (k & 1) * (32 * T);
        double* colb = rowb + 16 * T;
        if (ti == k0 / T) {
#pragma unroll
          for (int b = 0; b < T; b++) rowb[tj * T + b] = r[kk][b];
        }
        if (tj == k0 / T) {
#pragma unroll
          for (int a = 0; a < T; a++) colb[ti * T + a] = r[a][kk];
        }
        __syncthreads();
        double piv = rowb[k];
        if (!(piv * want_sign > 0.0)) { flag = true; piv = want_sign; }
        const double d = 1.0 / piv;
        double rs[T], cs[T];
#pragma unroll
        for (int b = 0; b < T; b++) rs[b] = rowb[tj * T + b] * d;
#pragma unroll
        for (int a = 0; a < T; a++) cs[a] = colb[ti * T + a];
        // rank-one step on the whole block; the pivot row and column (meaningless after it) are rewritten by their owners
#pragma unroll
        for (int a = 0; a < T; a++)
#pragma unroll
          for (int b = 0; b < T; b++) r[a][b] -= cs[a] * rs[b];
        if (tj == k0 / T) {
#pragma unroll
          for (int a = 0; a < T; a++) r[a][kk] = -cs[a] * d;
        }
        if (ti == k0 / T) {
#pragma unroll
          for (int b = 0; b < T; b++) r[kk][b] = rs[b];
          if (tj == k0 / T) r[kk][kk] = d;
        }
      }
    }
  }
  if (flag && tid == 0) *bad = 1;
#pragma unroll
  for (int a = 0; a < T; a++)
#pragma unroll
    for (int b = 0; b < T; b++) {
      const int i = ti * T + a, j = tj * T + b;
      if (i < n && j < n) A[i * n + j] = r[a][b];
    }
  __syncthreads();
}

constexpr int IB_LD = 17;
template <int NB> struct InvLds { double Pn[2][NB][16][IB_LD], Q[NB][16][IB_LD], D[2][16][IB_LD]; };
// Inverse of the symmetric positive definite w x w block that get(i, j), j <= i < w, returns (w <= 16 NB, NB <= W), by one
// workgroup of W waves that hold T of the lower 16 x 16 tiles each (W T >= NB (NB + 1) / 2); put(i, j, v), j <= i, receives it.
// The symmetric sweep 16 pivots at a time: the tiles of tile column kb go to LDS as P, Q = P D on the matrix cores, every
// other tile takes -= Q P^T, tile column kb becomes Q and its diagonal tile -D, so that the negated block is the inverse at
// the end.  What bounds it is the chain of pivots (one wave, about 0.1 us each; 256 threads with one pivot per barrier took
// 1.1 us each for 128 rows), so the wave that owns the next diagonal tile updates that one first and inverts it while the
// other waves finish their tiles.  A pivot that is not positive is taken as 1 and reported (by every lane).
template <int W, int T, int NB, typename Get, typename Put>
__device__ __forceinline__ bool inv_sym(int w, InvLds<NB>& L, Get get, Put put) {
  static_assert(NB <= W && W * T >= NB * (NB + 1) / 2, "tiles per wave");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const int nb = (w + 15) / 16;
  int ti[T], tj[T];
  swd4 x[T];
  bool flag = false;
#pragma unroll
  for (int s = 0; s < T; s++) {
    const int t = wave + W * s;
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= t) I++;
    ti[s] = __builtin_amdgcn_readfirstlane(I); tj[s] = __builtin_amdgcn_readfirstlane(t - I * (I + 1) / 2);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = ti[s] * 16 + 4 * r + lr, j = tj[s] * 16 + lc;
      const int hi = i > j ? i : j, lo = i > j ? j : i;
      const double v = get(hi < w ? hi : w - 1, lo < w ? lo : w - 1);      // (a load under a condition is waited for by itself)
      x[s][r] = hi < w ? v : (i == j ? 1.0 : 0.0);
    }
  }
  auto invert = [&](const swd4& a, int kb) {
    swd4 y = a;
    inv16(y, lane, w - kb * 16, flag);
#pragma unroll
    for (int r = 0; r < 4; r++) L.D[kb & 1][4 * r + lr][lc] = y[r];
  };
  if (wave == 0) invert(x[0], 0);
  for (int kb = 0; kb < nb; kb++) {
    double (*P)[16][IB_LD] = L.Pn[kb & 1];
    double (*Dk)[IB_LD] = L.D[kb & 1];
#pragma unroll
    for (int s = 0; s < T; s++) {
      if (ti[s] >= nb) continue;
      if (tj[s] == kb && ti[s] > kb) {
#pragma unroll
        for (int r = 0; r < 4; r++) P[ti[s]][4 * r + lr][lc] = x[s][r];
      } else if (ti[s] == kb && tj[s] < kb) {
#pragma unroll
        for (int r = 0; r < 4; r++) P[tj[s]][lc][4 * r + lr] = x[s][r];
      }
    }
    __syncthreads();
    if (wave < nb && wave != kb) {
      swd4 q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 4; kk++)
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(P[wave][lc][kk * 4 + lr], Dk[kk * 4 + lr][lc], q, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; r++) L.Q[wave][4 * r + lr][lc] = q[r];
    }
    __syncthreads();
    auto update = [&](int s) {
      const int I = ti[s], J = tj[s];
      if (I >= nb) return;
      if (I != kb && J != kb) {
#pragma unroll
        for (int kk = 0; kk < 4; kk++)
          x[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(-L.Q[I][lc][kk * 4 + lr], P[J][lc][kk * 4 + lr], x[s], 0, 0, 0);
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++)
          x[s][r] = I > kb ? L.Q[I][4 * r + lr][lc] : J < kb ? L.Q[J][lc][4 * r + lr] : -Dk[4 * r + lr][lc];
      }
    };
#pragma unroll
    for (int s = 0; s < T; s++)
      if (ti[s] == kb + 1 && tj[s] == kb + 1 && kb + 1 < nb) { update(s); invert(x[s], kb + 1); }
#pragma unroll
    for (int s = 0; s < T; s++)
      if (!(ti[s] == kb + 1 && tj[s] == kb + 1)) update(s);
  }
#pragma unroll
  for (int s = 0; s < T; s++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = ti[s] * 16 + 4 * r + lr, j = tj[s] * 16 + lc;
      if (i < w && j <= i) put(i, j, -x[s][r]);
    }
  return __any(flag);
}

// out(i, j, sum_k a(i, k) b(k, j)) for i, j, k < q <= 16 RT, by the four waves of a workgroup, 16 x 16 tiles on the float64 matrix
// cores; a and b return float64 from wherever they lie.
template <int RT, typename FA, typename FB, typename FO>
__device__ __forceinline__ void mm_small(int q, FA a, FB b, FO out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
  for (int t = wave; t < RT * RT; t += 4) {
    const int i0 = t / RT * 16, j0 = t % RT * 16;
    if (i0 >= q || j0 >= q) continue;
    swd4 acc = {0.0, 0.0, 0.0, 0.0};
    const int ia = min(i0 + lc, q - 1), jb = min(j0 + lc, q - 1);      // rows and columns past the end are dropped
#pragma unroll 4
    for (int k0 = 0; k0 < q; k0 += 4) {
      const int k = k0 + lr, kc = min(k, q - 1);
      const double at = a(ia, kc), bt = b(kc, jb), av = k < q ? at : 0.0, bv = k < q ? bt : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; r++)
      if (i0 + 4 * r + lr < q && j0 + lc < q) out(i0 + 4 * r + lr, j0 + lc, acc[r]);
  }
}
// f(integral_constant RT) for the number of 16-row tiles of a group
#define OSSCAR_BY_TILES(q_, CALL)                                                        \
  switch (((q_) + 15) / 16) {                                                            \
    case 1: { constexpr int RT = 1; CALL; } break;                                       \
    case 2: { constexpr int RT = 2; CALL; } break;                                       \
    case 3: { constexpr int RT = 3; CALL; } break;                                       \
    default: { constexpr int RT = 4; CALL; } break;                                      \
  }

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

__device__ __forceinline__ float nsym(const float* __restrict__ N, int64_t ld, int i, int t) {
  return (i >= t) ? N[(int64_t)i * ld + t] : N[(int64_t)t * ld + i];
}

// ------------------------------------------------------------------------------------------------
// gather / scatter / mirror / absmax
// ------------------------------------------------------------------------------------------------
__global__ void gather_kernel(const float* __restrict__ src, int64_t lds_, const int32_t* __restrict__ rows, int nrows,
                              const int32_t* __restrict__ cols, int ncols, float* __restrict__ dst, int64_t ldd) {
  int64_t n = (int64_t)nrows * ncols;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / ncols), j = (int)(idx % ncols);
    int64_t r = rows ? rows[i] : i, c = cols ? cols[j] : j;
    dst[(int64_t)i * ldd + j] = src[r * lds_ + c];
  }
}
hipError_t launch_gather(const float* src, int64_t lds_, const int32_t* rows, int nrows, const int32_t* cols, int ncols,
                         float* dst, int64_t ldd, hipStream_t s) {
  int64_t n = (int64_t)nrows * ncols;
  if (n <= 0) return hipSuccess;
  int blocks = (int)((n + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(gather_kernel, dim3(blocks), dim3(256), 0, s, src, lds_, rows, nrows, cols, ncols, dst, ldd);
  return hipGetLastError();
}

// dst[max(r,c)][min(r,c)] = sign * src[i][j], r = rows[i], c = cols[j]; if tri: only i >= j
__global__ void scatter_kernel(const float* __restrict__ src, int64_t lds_, const int32_t* __restrict__ rows, int nrows,
                               const int32_t* __restrict__ cols, int ncols, float* __restrict__ dst, int64_t ldd,
                               float sign, int tri) {
  int64_t n = (int64_t)nrows * ncols;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / ncols), j = (int)(idx % ncols);
    if (tri && i < j) continue;
    int64_t r = rows[i], c = cols[j];
    int64_t hi = r > c ? r : c, lo = r > c ? c : r;
    dst[hi * ldd + lo] = sign * src[(int64_t)i * lds_ + j];
  }
}
hipError_t launch_scatter(const float* src, int64_t lds_, const int32_t* rows, int nrows, const int32_t* cols, int ncols,
                          float* dst, int64_t ldd, float sign, int tri, hipStream_t s) {
  int64_t n = (int64_t)nrows * ncols;
  if (n <= 0) return hipSuccess;
  int blocks = (int)((n + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks), dim3(256), 0, s, src, lds_, rows, nrows, cols, ncols, dst, ldd, sign, tri);
  return hipGetLastError();
}

// rows of a dense matrix into rows[] of dst (float or bf16 destination)
__device__ __forceinline__ uint16_t float_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__global__ void scatter_rows_kernel(const float* __restrict__ src, int64_t lds_, const int32_t* __restrict__ rows,
                                    int nrows, int ncols, void* __restrict__ dst, int64_t ldd, int dst_is_bf16) {
  int64_t n = (int64_t)nrows * ncols;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / ncols), j = (int)(idx % ncols);
    float v = src[(int64_t)i * lds_ + j];
    int64_t o = (int64_t)rows[i] * ldd + j;
    if (dst_is_bf16) reinterpret_cast<uint16_t*>(dst)[o] = float_to_bf16_rne(v);
    else reinterpret_cast<float*>(dst)[o] = v;
  }
}
hipError_t launch_scatter_rows(const float* src, int64_t lds_, const int32_t* rows, int nrows, int ncols, void* dst,
                               int64_t ldd, int dst_is_bf16, hipStream_t s) {
  int64_t n = (int64_t)nrows * ncols;
  if (n <= 0) return hipSuccess;
  int blocks = (int)((n + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(scatter_rows_kernel, dim3(blocks), dim3(256), 0, s, src, lds_, rows, nrows, ncols, dst, ldd, dst_is_bf16);
  return hipGetLastError();
}
__global__ void fill_zero_kernel(void* __restrict__ dst, int64_t ldd, int nrows, int ncols, int dst_is_bf16) {
  int64_t n = (int64_t)nrows * ncols;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / ncols), j = (int)(idx % ncols);
    int64_t o = (int64_t)i * ldd + j;
    if (dst_is_bf16) reinterpret_cast<uint16_t*>(dst)[o] = 0;
    else reinterpret_cast<float*>(dst)[o] = 0.f;
  }
}
hipError_t launch_fill_rows_zero(void* dst, int64_t ldd, int nrows, int ncols, int dst_is_bf16, hipStream_t s) {
  int64_t n = (int64_t)nrows * ncols;
  if (n <= 0) return hipSuccess;
  int blocks = (int)((n + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, dst, ldd, nrows, ncols, dst_is_bf16);
  return hipGetLastError();
}

// A[i][j] (j > i) = A[j][i]
__global__ void mirror_lower_kernel(float* __restrict__ A, int n, int64_t lda) {
  int64_t tot = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / n), j = (int)(idx % n);
    if (j > i) A[(int64_t)i * lda + j] = A[(int64_t)j * lda + i];
  }
}
hipError_t launch_mirror_lower(float* A, int n, int64_t lda, hipStream_t s) {
  int64_t tot = (int64_t)n * n;
  if (tot <= 0) return hipSuccess;
  int blocks = (int)((tot + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(mirror_lower_kernel, dim3(blocks), dim3(256), 0, s, A, n, lda);
  return hipGetLastError();
}

// out[b] for 256 blocks, then the caller reduces on the host (256 doubles).  A bandwidth-bound pass: 1024 threads per
// block, four 16-byte loads in flight per thread (scalar loads for an unaligned start and for the tail).
__device__ __forceinline__ float absmax_take(float v, float x) { x = fabsf(x); return (x > v || x != x) ? x : v; }
__global__ __launch_bounds__(1024) void absmax_partial_kernel(const float* __restrict__ A, int64_t n, double* out) {
  __shared__ float sh[16];
  // a NaN is taken (x != x) and then stays (nothing compares greater than it), so a NaN anywhere reaches the result
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  const int64_t head = ((reinterpret_cast<uintptr_t>(A) & 15) == 0) ? 0 : n;      // unaligned: everything in the scalar loop
  const int64_t n4 = (n - head) / 4;
  const float4* A4 = reinterpret_cast<const float4*>(A);
  const int64_t tid = blockIdx.x * 1024 + threadIdx.x, nth = (int64_t)gridDim.x * 1024;
  for (int64_t i = tid; i < n4; i += 4 * nth) {
    float4 q[4];
#pragma unroll
    for (int u = 0; u < 4; u++) { const int64_t k = i + u * nth; q[u] = A4[k < n4 ? k : i]; }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      v[u] = absmax_take(v[u], q[u].x); v[u] = absmax_take(v[u], q[u].y); v[u] = absmax_take(v[u], q[u].z); v[u] = absmax_take(v[u], q[u].w);
    }
  }
  for (int64_t i = head == 0 ? 4 * n4 + tid : tid; i < n; i += nth) v[0] = absmax_take(v[0], A[i]);
  float t = v[0];
#pragma unroll
  for (int u = 1; u < 4; u++) t = (v[u] > t || v[u] != v[u]) ? v[u] : t;
  for (int o = 32; o > 0; o >>= 1) { const float w = __shfl_down(t, o, 64); t = (w > t || w != w) ? w : t; }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) { float r = 0.f; for (int i = 0; i < 16; i++) r = (sh[i] > r || sh[i] != sh[i]) ? sh[i] : r; out[blockIdx.x] = (double)r; }
}
hipError_t launch_absmax(const float* A, int64_t n, double* out, hipStream_t s) {  // out: 256 doubles
  hipLaunchKernelGGL(absmax_partial_kernel, dim3(256), dim3(1024), 0, s, A, n, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// pivot panels
// ------------------------------------------------------------------------------------------------
// C[i][c] = Nsym(i, t0 + c), c < w <= 128, for all rows i < n.  One workgroup per 64 rows: below the pivot rows the panel
// is a column block of N (read along c); above them it lies transposed in the rows t0 + c of N (read along i and turned
// in shared memory); the few blocks that meet the pivot rows take either side element by element.
constexpr int PANEL_ROWS = 64;
__global__ __launch_bounds__(256) void extract_panel_kernel(const float* __restrict__ N, int64_t ld, int n, int t0,
                                                             int w, float* __restrict__ C) {
  __shared__ float T[PANEL_ROWS][129];
  const int i0 = blockIdx.x * PANEL_ROWS, tid = threadIdx.x;
  if (i0 >= t0 + w) {
    for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
      const int r = idx / w, c = idx % w;
      if (i0 + r < n) C[(int64_t)(i0 + r) * w + c] = N[(int64_t)(i0 + r) * ld + t0 + c];
    }
    return;
  }
  if (i0 + PANEL_ROWS <= t0) {
    for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
      const int c = idx / PANEL_ROWS, r = idx % PANEL_ROWS;
      T[r][c] = N[(int64_t)(t0 + c) * ld + i0 + r];
    }
  } else {
    for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
      const int r = idx / w, c = idx % w;
      T[r][c] = (i0 + r < n) ? nsym(N, ld, i0 + r, t0 + c) : 0.f;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
    const int r = idx / w, c = idx % w;
    if (i0 + r < n) C[(int64_t)(i0 + r) * w + c] = T[r][c];
  }
}

// out[i][c] = sum_k C[i][k] * D[k][c]  (D: w x w float64, w <= 128), rows in [t0, t0+w) are written as zero if zero_pivot.
// Optionally also writes Cb = C with the pivot rows zeroed.  16 rows per workgroup: their C values are broadcast from
// LDS, thread (h, c) sums 8 rows of column c in float64, k ascending.
__global__ __launch_bounds__(256) void panel_times_small_kernel(const float* __restrict__ C, const double* __restrict__ D,
                                                                 int n, int w, int t0, int zero_pivot,
                                                                 float* __restrict__ out, float* __restrict__ Cb) {
  __shared__ float Csh[16][128];
  const int r0 = blockIdx.x * 16, tid = threadIdx.x;
  for (int idx = tid; idx < 16 * w; idx += 256) {
    const int r = idx / w, k = idx % w;
    Csh[r][k] = (r0 + r < n) ? C[(int64_t)(r0 + r) * w + k] : 0.f;
  }
  __syncthreads();
  const int c = tid & 127, h = tid >> 7;
  if (c >= w) return;
  double acc[8];
#pragma unroll
  for (int r = 0; r < 8; r++) acc[r] = 0.0;
  for (int k = 0; k < w; k++) {
    const double dv = D[k * w + c];
#pragma unroll
    for (int r = 0; r < 8; r++) acc[r] += (double)Csh[h * 8 + r][k] * dv;
  }
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int i = r0 + h * 8 + r;
    if (i >= n) continue;
    const bool piv = zero_pivot && i >= t0 && i < t0 + w;
    out[(int64_t)i * w + c] = piv ? 0.f : (float)acc[r];
    if (Cb) Cb[(int64_t)i * w + c] = piv ? 0.f : Csh[h * 8 + r][c];
  }
}

// ------------------------------------------------------------------------------------------------
// blocked in-place inverse of an SPD matrix by sweeping nb columns at a time (lower triangle storage)
// ------------------------------------------------------------------------------------------------
// D = inverse of the w x w pivot block (rows t0.. of the extracted panel), float64
__global__ __launch_bounds__(256) void inv_block_kernel(const float* __restrict__ C, int w, int t0, double* __restrict__ D,
                                                         int32_t* notpd) {
  __shared__ double buf[64 * (INV_NB / 16)];
  for (int idx = threadIdx.x; idx < w * w; idx += 256) {
    int r = idx / w, c = idx % w;
    D[idx] = (double)C[(int64_t)(t0 + r) * w + c];
  }
  small_inverse<INV_NB / 16>(D, w, +1, notpd, buf);
}

// pivot rows after a forward sweep: N(t0+r, l) = CD[l][r] for l outside the pivot, N(tt) = -D
__global__ __launch_bounds__(256) void inv_fix_kernel(float* __restrict__ N, int64_t ld, int n, int t0, int w,
                                                       const float* __restrict__ CD, const double* __restrict__ D) {
  __shared__ float T[PANEL_ROWS][129];
  const int i0 = blockIdx.x * PANEL_ROWS, tid = threadIdx.x;
  if (i0 >= t0 + w) {                         // below the pivot rows: a column block of N
    for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
      const int r = idx / w, c = idx % w;
      if (i0 + r < n) N[(int64_t)(i0 + r) * ld + t0 + c] = CD[(int64_t)(i0 + r) * w + c];
    }
    return;
  }
  for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
    const int r = idx / w, c = idx % w;
    T[r][c] = (i0 + r < n) ? CD[(int64_t)(i0 + r) * w + c] : 0.f;
  }
  __syncthreads();
  if (i0 + PANEL_ROWS <= t0) {                // above: the rows t0 + c of N, written along i
    for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {
      const int c = idx / PANEL_ROWS, r = idx % PANEL_ROWS;
      N[(int64_t)(t0 + c) * ld + i0 + r] = T[r][c];
    }
    return;
  }
  for (int idx = tid; idx < PANEL_ROWS * w; idx += 256) {     // a block that meets the pivot rows
    const int r = idx / w, c = idx % w, l = i0 + r;
    if (l >= n) continue;
    if (l < t0) N[(int64_t)(t0 + c) * ld + l] = T[r][c];
    else if (l >= t0 + w) N[(int64_t)l * ld + t0 + c] = T[r][c];
    else if (c <= l - t0) N[(int64_t)l * ld + t0 + c] = (float)(-D[(l - t0) * w + c]);
  }
}

// A[i][j] = -A[max][min] for all i, j (turns the swept lower triangle -A^-1 into the full inverse)
__global__ void negate_mirror_kernel(float* __restrict__ A, int n) {
  int64_t tot = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / n), j = (int)(idx % n);
    if (j <= i) continue;
    float v = -A[(int64_t)j * n + i];
    A[(int64_t)i * n + j] = v;     // upper gets the final value
  }
}
__global__ void negate_lower_kernel(float* __restrict__ A, int n) {
  int64_t tot = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / n), j = (int)(idx % n);
    if (j <= i) A[idx] = -A[idx];
  }
}

hipError_t spd_inverse_inplace(float* A, int n, float* panel, float* panelD, double* small, int32_t* notpd_flag,
                               hipStream_t s) {
  float* panelB = panelD + (int64_t)n * INV_NB;   // caller provides 2*n*nb floats behind panelD
  for (int t0 = 0; t0 < n; t0 += INV_NB) {
    int w = (n - t0 < INV_NB) ? n - t0 : INV_NB;
    int rb = (n + PANEL_ROWS - 1) / PANEL_ROWS;
    hipLaunchKernelGGL(extract_panel_kernel, dim3(rb), dim3(256), 0, s, A, (int64_t)n, n, t0, w, panel);
    hipLaunchKernelGGL(inv_block_kernel, dim3(1), dim3(256), 0, s, panel, w, t0, small, notpd_flag);
    // true C*D for the pivot-row fix, and zeroed copies for the bulk update
    hipLaunchKernelGGL(panel_times_small_kernel, dim3((n + 15) / 16), dim3(256), 0, s, panel, small, n, w, t0, 1, panelD,
                       panelB);
    GemmArgs g{};
    g.M = n; g.N = n; g.K = w; g.A = panelD; g.lda = w; g.B = panelB; g.ldb = w; g.trans_b = 1;
    g.Cin = A; g.ldcin = n; g.C = A; g.ldc = n; g.alpha = -1.0; g.beta = 1.0; g.diag_add = 0.0; g.c_is_f64 = 0;
    g.lower_only = 1; g.acc_f32 = 1;
    hipError_t e = launch_gemm_f64acc(g, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(inv_fix_kernel, dim3(rb), dim3(256), 0, s, A, (int64_t)n, n, t0, w, panelD, small);
  }
  int64_t tot = (int64_t)n * n;
  int blocks = (int)((tot + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(negate_mirror_kernel, dim3(blocks), dim3(256), 0, s, A, n);
  hipLaunchKernelGGL(negate_lower_kernel, dim3(blocks), dim3(256), 0, s, A, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The same blocked sweep with the working matrix held in float64.  In float32 storage every one of the n / 128 panel
// updates rounds every entry again, and the inverse comes out with |I - H P| of 1e-5: it then needs a Newton-Schulz step
// whose residual I - H P is a full n^3 product with float64 sums (93 ms for n = 14336, a third of the state build).  Held
// in float64 the swept matrix is exact to 1e-12 and is rounded to float32 once: the same accuracy as after that step, for a
// rank-128 update that moves 16 bytes per entry instead of 8 (0.5 ms instead of 0.33 ms per panel).
// ------------------------------------------------------------------------------------------------
constexpr int PANEL_ROWS64 = 32;
__device__ __forceinline__ double nsym64(const double* __restrict__ N, int64_t ld, int i, int t) {
  return (i >= t) ? N[(int64_t)i * ld + t] : N[(int64_t)t * ld + i];
}
// A[i][j] = H[i][j] for j <= i (only the lower triangle is ever read)
__global__ void widen_lower_kernel(const float* __restrict__ H, int64_t ldh, int n, double* __restrict__ A) {
  const int64_t tot = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / n), j = (int)(idx % n);
    if (j <= i) A[idx] = (double)H[(int64_t)i * ldh + j];
  }
}
// P[i][j] = P[j][i] = float(-A[i][j]), j <= i: the swept lower triangle -H^-1 as the full float32 inverse.  One workgroup per
// 32 x 32 tile on or below the diagonal; the mirrored tile is written from shared memory so that both writes run along rows.
__global__ __launch_bounds__(256) void narrow_negate_mirror_kernel(const double* __restrict__ A, int n, float* __restrict__ P) {
  __shared__ float T[32][33];
  int bi = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
  while ((int64_t)(bi + 1) * (bi + 2) / 2 <= (int64_t)blockIdx.x) bi++;
  while ((int64_t)bi * (bi + 1) / 2 > (int64_t)blockIdx.x) bi--;
  const int bj = (int)(blockIdx.x - (int64_t)bi * (bi + 1) / 2);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int r = ty + 8 * k, i = bi * 32 + r, j = bj * 32 + tx;
    T[r][tx] = (i < n && j <= i) ? (float)(-A[(int64_t)i * n + j]) : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int r = ty + 8 * k;
    const int i = bi * 32 + r, j = bj * 32 + tx;
    if (i < n && j < n) {
      if (j <= i) P[(int64_t)i * n + j] = T[r][tx];
      else if (bi == bj) P[(int64_t)i * n + j] = T[tx][r];       // upper part of a diagonal tile
    }
    if (bi != bj) {
      const int mi = bj * 32 + r, mj = bi * 32 + tx;             // the mirrored tile, row r of it = column r of this one
      if (mi < n && mj < n) P[(int64_t)mi * n + mj] = T[tx][r];
    }
  }
}
// Cz = the pivot columns t0 .. t0 + w of N for every row but the pivot's own, which are zero there (an operand of the bulk update), and
// (the first workgroup) D = the inverse of the pivot block, straight from N, so that the copy runs beside the inverse.
constexpr int IB_T = 768;                              // 12 waves x 3 of the 36 lower tiles of a pivot block
__global__ __launch_bounds__(IB_T) void panel_inverse64_kernel(const double* __restrict__ N, int64_t ld, int n, int t0, int w,
                                                                double* __restrict__ C, double* __restrict__ D, int32_t* notpd) {
  __shared__ InvLds<8> L;
  static_assert(sizeof(InvLds<8>) >= PANEL_ROWS64 * 129 * sizeof(double), "the copy's tile shares the inverse's memory");
  if (blockIdx.x == 0) {
    const bool bad = inv_sym<12, 3, 8>(w, L, [&](int i, int j) { return N[(int64_t)(t0 + i) * ld + t0 + j]; },
                                       [&](int i, int j, double v) { D[i * w + j] = v; D[j * w + i] = v; });
    if (bad && (threadIdx.x & 63) == 0) *notpd = 1;
    return;
  }
  double (*T)[129] = reinterpret_cast<double (*)[129]>(&L);
  const int i0 = (blockIdx.x - 1) * PANEL_ROWS64, tid = threadIdx.x;
  if (i0 >= t0 + w) {
    for (int idx = tid; idx < PANEL_ROWS64 * w; idx += IB_T) {
      const int r = idx / w, c = idx % w;
      if (i0 + r < n) C[(int64_t)(i0 + r) * w + c] = N[(int64_t)(i0 + r) * ld + t0 + c];
    }
    return;
  }
  if (i0 + PANEL_ROWS64 <= t0) {
    for (int idx = tid; idx < PANEL_ROWS64 * w; idx += IB_T) {
      const int c = idx / PANEL_ROWS64, r = idx % PANEL_ROWS64;
      T[r][c] = N[(int64_t)(t0 + c) * ld + i0 + r];
    }
  } else {
    for (int idx = tid; idx < PANEL_ROWS64 * w; idx += IB_T) {
      const int r = idx / w, c = idx % w;
      const bool piv = i0 + r >= t0 && i0 + r < t0 + w;
      T[r][c] = (i0 + r < n && !piv) ? nsym64(N, ld, i0 + r, t0 + c) : 0.0;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < PANEL_ROWS64 * w; idx += IB_T) {
    const int r = idx / w, c = idx % w;
    if (i0 + r < n) C[(int64_t)(i0 + r) * w + c] = T[r][c];
  }
}
// outz = Cz D, the other operand, whose pivot rows are zero too (the pivot-row fix reads it outside them).  16 rows per workgroup on the float64 matrix
// cores, wave w: columns 32 w .. + 31; D is symmetric and comes from L2, eight steps of four requested ahead.  Bound by that latency (in scalars, with a
// pass over C in front, 10.5 us for 1536 rows and 53 for 8192).
__global__ __launch_bounds__(256) void panel_times_block64_kernel(const double* __restrict__ Cz, const double* __restrict__ D, int n, int w, double* __restrict__ outz) {
  __shared__ double As[16][130];
  const int r0 = blockIdx.x * 16, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  double c[8];
#pragma unroll
  for (int u = 0; u < 8; u++) {
    const int idx = tid + 256 * u, r = min(r0 + (idx >> 7), n - 1), k = min(idx & 127, w - 1);
    c[u] = Cz[(int64_t)r * w + k];
  }
  const int col0 = min(wave * 32 + lc, w - 1), col1 = min(wave * 32 + 16 + lc, w - 1);
  double d0[2][8], d1[2][8];
  auto request = [&](int g, double (&p)[8], double (&q)[8]) {
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const int64_t k = min(g * 32 + 4 * u + lr, w - 1);      // (past the end: times zero)
      p[u] = D[k * w + col0]; q[u] = D[k * w + col1];
    }
  };
  request(0, d0[0], d1[0]);
#pragma unroll
  for (int u = 0; u < 8; u++) {
    const int idx = tid + 256 * u;
    As[idx >> 7][idx & 127] = (idx & 127) < w ? c[u] : 0.0;
  }
  __syncthreads();
  swd4 acc[2] = {swd4{0.0, 0.0, 0.0, 0.0}, swd4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int g = 0; g < 4; g++) {
    if (g < 3) request(g + 1, d0[(g + 1) & 1], d1[(g + 1) & 1]);
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const double a = As[lc][g * 32 + 4 * u + lr];
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, d0[g & 1][u], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, d1[g & 1][u], acc[1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int i = r0 + 4 * r + lr;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int col = wave * 32 + 16 * j + lc;
      if (i < n && col < w) outz[(int64_t)i * w + col] = acc[j][r];
    }
  }
}
// pivot rows after the sweep of rows t0 .. t0 + w, for the 32 rows i0 ..: N(t0 + c, l) = CD[l][c] outside the pivot, -D on it
__device__ void inv_fix64(double* __restrict__ N, int64_t ld, int n, int t0, int w, const double* __restrict__ CD,
                          const double* __restrict__ D, int i0, double (*T)[129]) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (i0 >= t0 + w) {
    for (int idx = tid; idx < PANEL_ROWS64 * w; idx += nt) {
      const int r = idx / w, c = idx % w;
      if (i0 + r < n) N[(int64_t)(i0 + r) * ld + t0 + c] = CD[(int64_t)(i0 + r) * w + c];
    }
    return;
  }
  for (int idx = tid; idx < PANEL_ROWS64 * w; idx += nt) {
    const int r = idx / w, c = idx % w;
    T[r][c] = (i0 + r < n) ? CD[(int64_t)(i0 + r) * w + c] : 0.0;
  }
  __syncthreads();
  if (i0 + PANEL_ROWS64 <= t0) {
    for (int idx = tid; idx < PANEL_ROWS64 * w; idx += nt) {
      const int c = idx / PANEL_ROWS64, r = idx % PANEL_ROWS64;
      N[(int64_t)(t0 + c) * ld + i0 + r] = T[r][c];
    }
    return;
  }
  for (int idx = tid; idx < PANEL_ROWS64 * w; idx += nt) {
    const int r = idx / w, c = idx % w, l = i0 + r;
    if (l >= n) continue;
    if (l < t0) N[(int64_t)(t0 + c) * ld + l] = T[r][c];
    else if (l >= t0 + w) N[(int64_t)l * ld + t0 + c] = T[r][c];
    else if (c <= l - t0) N[(int64_t)l * ld + t0 + c] = -D[(l - t0) * w + c];
  }
}

// N[i][j] -= sum_k A[i][k] B[j][k] on the tiles of the lower block triangle; A, B: n x w float64 (w <= 128), N: n x n float64.
// One workgroup per half (128 rows x 64 columns) of a 128 x 128 tile, 8 waves x (2 x 2) v_mfma_f64_16x16x4_f64, the
// contraction in steps of 16 through LDS (rows of 144 and 80 doubles: the four k of a quarter-wave's operand read fall in
// different bank groups).  The workgroup's part of N (16 values per thread) is requested while the first products run and is
// there when the last one ends: with a whole tile per workgroup the registers held a quarter of it at a time, and four
// round trips to memory followed the products.  Tiles in 8 x 8 super-blocks per XCD, the two halves of a tile on one XCD.
constexpr int SW_LD = 144, SW_LDB = 80;
constexpr size_t SW_LDS_BYTES = (size_t)2 * 16 * (SW_LD + SW_LDB) * sizeof(double);
// part = 0: every tile of the triangle.  The pivot rows of A and B are zero, so the tiles of tile row / column pk (the
// pivot panel's) receive nothing and are always left alone (the pivot-row fix rewrites them, possibly meanwhile).
// part = 1: only tile row and tile column pk + 1, what the next panel is made of (two workgroups per tile, blockIdx / 2 =
// the other tile index); part = 2: everything but those.
// Workgroups from fix_at on write the pivot rows instead (32 rows each; D = the inverse of the pivot block): they touch
// tile row and column pk only, and as a launch of their own behind part 1 they cost the next panel 10 - 15 us.
__global__ __launch_bounds__(512, 2) void sweep_update64_kernel(const double* __restrict__ A, const double* __restrict__ B, int n, int w,
                                                                 double* __restrict__ N, int part, int pk, unsigned fix_at,
                                                                 const double* __restrict__ D) {
  extern __shared__ double sw_lds[];           // 56 KB: above the static limit, so taken dynamically
  if (blockIdx.x >= fix_at) {
    inv_fix64(N, n, n, pk * INV_NB, w, A, D, (int)(blockIdx.x - fix_at) * PANEL_ROWS64, reinterpret_cast<double (*)[129]>(sw_lds));
    return;
  }
  double (*As)[16][SW_LD] = reinterpret_cast<double (*)[16][SW_LD]>(sw_lds);
  double (*Bs)[16][SW_LDB] = reinterpret_cast<double (*)[16][SW_LDB]>(sw_lds + 2 * 16 * SW_LD);
  int tm, tn, half;
  if (part == 1) {
    const int tiles = (n + 127) / 128, b = blockIdx.x >> 1, nx = pk + 1;
    half = blockIdx.x & 1;
    if (b >= tiles || nx >= tiles || b == pk) return;
    tm = (b <= nx) ? nx : b;
    tn = (b <= nx) ? b : nx;
  } else {
    const int tiles = (n + 127) / 128, nr = (tiles + 7) / 8;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 4;
    half = (blockIdx.x >> 3) & 1;
    const int sb = (slot / 64) * 8 + xcd, within = slot % 64;
    if (sb >= nr * (nr + 1) / 2) return;
    int r = (int)((sqrtf(8.f * (float)sb + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= sb) r++;
    while (r * (r + 1) / 2 > sb) r--;
    tm = r * 8 + within / 8;
    tn = (sb - r * (r + 1) / 2) * 8 + within % 8;
    if (tm >= tiles || tn > tm) return;
    if (tm == pk || tn == pk) return;
    if (part == 2 && (tm == pk + 1 || tn == pk + 1)) return;
  }
  const int m0 = tm * 128, n0 = tn * 128 + half * 64;
  if (n0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;   // wave tile: 32 rows x 32 columns
  const int lrow = tid >> 2, lk = (tid & 3) * 4;        // staging: thread = (row of the tile, quarter of the 16 k)
  const bool stage_b = lrow < 64;                       // B has 64 rows here
  const double* ap = (m0 + lrow < n) ? A + (int64_t)(m0 + lrow) * w : nullptr;
  const double* bp = (stage_b && n0 + lrow < n) ? B + (int64_t)(n0 + lrow) * w : nullptr;
  swd4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) acc[i][j] = swd4{0.0, 0.0, 0.0, 0.0};
  double ra[4], rb[4];
  const int ktiles = (w + 15) / 16;
  const bool vec = (w & 3) == 0;       // then a thread's four k are inside or outside as a whole, and 32-byte aligned
  auto gload = [&](int kt) {
    const int k0 = kt * 16 + lk;
    if (vec) {
      if (ap && k0 < w) {
        const double2* p = reinterpret_cast<const double2*>(ap + k0);
        const double2 q0 = p[0], q1 = p[1];
        ra[0] = q0.x; ra[1] = q0.y; ra[2] = q1.x; ra[3] = q1.y;
      } else { ra[0] = ra[1] = ra[2] = ra[3] = 0.0; }
      if (bp && k0 < w) {
        const double2* p = reinterpret_cast<const double2*>(bp + k0);
        const double2 q0 = p[0], q1 = p[1];
        rb[0] = q0.x; rb[1] = q0.y; rb[2] = q1.x; rb[3] = q1.y;
      } else { rb[0] = rb[1] = rb[2] = rb[3] = 0.0; }
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int k = k0 + e;
      ra[e] = (ap && k < w) ? ap[k] : 0.0;
      rb[e] = (bp && k < w) ? bp[k] : 0.0;
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int e = 0; e < 4; e++) As[buf][lk + e][lrow] = ra[e];
    if (stage_b) {
#pragma unroll
      for (int e = 0; e < 4; e++) Bs[buf][lk + e][lrow] = rb[e];
    }
  };
  // lane holds D[4 r + lane/16][lane%16] of each 16 x 16 tile
  const int rbase = m0 + wm * 32 + (lane >> 4), cbase = n0 + wn * 32 + (lane & 15);
  const bool whole = (m0 + 128 <= n && n0 + 64 <= n);
  double* nbase = N + (int64_t)rbase * n + cbase;       // dereferenced only where the row and column exist
  double cv[2][2][4];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) cv[i][j][r] = 0.0;
  if (ktiles > 0) { gload(0); sstore(0); }
  __syncthreads();
  if (whole && w == 128) {
    // The usual case.  The 16 values of N are requested two per stage, each pair behind the next stage's operands: the wait
    // for those operands at the end of a stage then covers the pair requested a stage earlier, and the requests to memory
    // run through the whole contraction instead of piling up at its start.
#pragma unroll
    for (int kt = 0; kt < 8; kt++) {
      const int buf = kt & 1;
      if (kt + 1 < 8) gload(kt + 1);
#pragma unroll
      for (int e = kt * 2; e < kt * 2 + 2; e++)
        cv[e >> 3][(e >> 2) & 1][e & 3] = nbase[(int64_t)((e >> 3) * 16 + 4 * (e & 3)) * n + ((e >> 2) & 1) * 16];
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        const int k = kk * 4 + (lane >> 4);
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; i++) a[i] = As[buf][k][wm * 32 + i * 16 + (lane & 15)];
#pragma unroll
        for (int j = 0; j < 2; j++) b[j] = Bs[buf][k][wn * 32 + j * 16 + (lane & 15)];
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      if (kt + 1 < 8) sstore(buf ^ 1);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) nbase[(int64_t)(i * 16 + 4 * r) * n + j * 16] = cv[i][j][r] - acc[i][j][r];
    return;
  }
  for (int kt = 0; kt < ktiles; kt++) {
    const int buf = kt & 1;
    if (kt + 1 < ktiles) gload(kt + 1);
    if (kt == 0) {
      // requested behind the second stage's operands, so that no operand load queues up behind them before they are back
      if (whole) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) cv[i][j][r] = nbase[(int64_t)(i * 16 + 4 * r) * n + j * 16];
      } else {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
              const int row = rbase + i * 16 + 4 * r, col = cbase + j * 16;
              cv[i][j][r] = (row < n && col < n) ? N[(int64_t)row * n + col] : 0.0;
            }
      }
    }
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      const int k = kk * 4 + (lane >> 4);
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; i++) a[i] = As[buf][k][wm * 32 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 2; j++) b[j] = Bs[buf][k][wn * 32 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < ktiles) sstore(buf ^ 1);
    __syncthreads();
  }
  if (ktiles == 0) return;
  if (whole) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) nbase[(int64_t)(i * 16 + 4 * r) * n + j * 16] = cv[i][j][r] - acc[i][j][r];
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int row = rbase + i * 16 + 4 * r, col = cbase + j * 16;
        if (row < n && col < n) N[(int64_t)row * n + col] = cv[i][j][r] - acc[i][j][r];
      }
}

// P (n x n float32, full) = H^-1 for the SPD H (n x n float32, leading dimension ldh; only its lower triangle is read).
// A64: n x n float64 work matrix; panels: 4 n INV_NB float64; small: INV_NB^2 float64; notpd_flag as for spd_inverse_inplace.
// With a side stream the panel work of step k + 1 (extract, 128 x 128 inverse, panel x block: 0.2 ms during which one
// workgroup, then a few, have the chip to themselves) runs beside the bulk update of step k: the tiles the next panel is made
// of (tile row and column k + 1) are updated first by a launch of their own, the pivot rows of step k are fixed, and the
// rest of the update goes to the side stream.  Each tile sees the same operations in the same order either way.
hipError_t spd_inverse_f64(const float* H, int64_t ldh, int n, float* P, double* A64, double* panels, double* small,
                           int32_t* notpd_flag, hipStream_t s, const SideStream* side) {
  if (n <= 0) return hipSuccess;
  const int64_t tot = (int64_t)n * n;
  int blocks = (int)((tot + 1023) / 1024); if (blocks > 131072) blocks = 131072;
  hipLaunchKernelGGL(widen_lower_kernel, dim3(blocks), dim3(256), 0, s, H, ldh, n, A64);
  const size_t shmem = SW_LDS_BYTES;
  {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(sweep_update64_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return e;
  }
  const int tiles = (n + 127) / 128, nr = (tiles + 7) / 8;
  const unsigned upd_grid = (unsigned)((nr * (nr + 1) / 2 + 7) / 8 * 8 * 64) * 2;      // two workgroups per tile
  const int rb = (n + PANEL_ROWS64 - 1) / PANEL_ROWS64;
  // (up to ten tiles a side the whole update takes as long as the next panel's part of it: 1152 rows 0.66 ms in order, 0.69 on two streams;
  // 2048 rows 1.43 and 1.25)
  const bool two = side && side->stream && tiles > 10;
  hipError_t err;
  bool pending = false;              // a bulk update is running on the side stream
  for (int t0 = 0, k = 0; t0 < n; t0 += INV_NB, k++) {
    const int w = (n - t0 < INV_NB) ? n - t0 : INV_NB;
    // operand panels alternate: the bulk update of step k - 1 may still be reading the other pair
    double* panelDz = panels + (int64_t)(2 * (k & 1)) * n * INV_NB;
    double* panelCz = panelDz + (int64_t)n * INV_NB;
    hipLaunchKernelGGL(panel_inverse64_kernel, dim3(rb + 1), dim3(IB_T), 0, s, A64, (int64_t)n, n, t0, w, panelCz, small, notpd_flag);
    hipLaunchKernelGGL(panel_times_block64_kernel, dim3((n + 15) / 16), dim3(256), 0, s, panelCz, small, n, w, panelDz);
    if (!two) {
      hipLaunchKernelGGL(sweep_update64_kernel, dim3(upd_grid + rb), dim3(512), shmem, s, panelDz, panelCz, n, w, A64, 0, k, upd_grid, small);
      continue;
    }
    // The bulk updates follow one another on the side stream without a gap: step k's needs its operands (ready here) and
    // step k - 1 on every tile it touches (the stream's order), nothing from this stream's later work.
    if ((err = hipEventRecord(side->fork, s)) != hipSuccess) return err;
    if ((err = hipStreamWaitEvent(side->stream, side->fork, 0)) != hipSuccess) return err;
    // This stream's next launch changes the next panel's tiles, which the bulk update of step k - 1 also does: it waits for
    // that one (the event's latest record), not for step k's, whose launch leaves those tiles out.
    if (pending && (err = hipStreamWaitEvent(s, side->join, 0)) != hipSuccess) return err;
    hipLaunchKernelGGL(sweep_update64_kernel, dim3(upd_grid), dim3(512), shmem, side->stream, panelDz, panelCz, n, w, A64, 2, k, upd_grid, small);
    if ((err = hipEventRecord(side->join, side->stream)) != hipSuccess) return err;
    pending = true;
    // with the pivot rows of this step: tile row and column k only, which no launch of this step's update touches and the next
    // step's bulk update does (it is enqueued behind an event that this stream records later)
    const unsigned next = k + 1 < tiles ? 2u * tiles : 0u;
    hipLaunchKernelGGL(sweep_update64_kernel, dim3(next + rb), dim3(512), shmem, s, panelDz, panelCz, n, w, A64, 1, k, next, small);
  }
  if (pending && (err = hipStreamWaitEvent(s, side->join, 0)) != hipSuccess) return err;
  const int64_t t32 = (n + 31) / 32;
  hipLaunchKernelGGL(narrow_negate_mirror_kernel, dim3((unsigned)(t32 * (t32 + 1) / 2)), dim3(256), 0, s, A64, n, P);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// scores: gram[h] = Z_h Z_h^T, dblk[h] = N_hh (float64), score[h] = Tr(gram_h |N_hh|^-1)
// ------------------------------------------------------------------------------------------------
// groups of one row: gram[h] = |Z_h|^2 and dblk[h] = N_hh, one wave per row (four rows per workgroup), 16-byte loads
__global__ __launch_bounds__(256) void gram_dblk_q1_kernel(int d1, int m, const float* __restrict__ N, const float* __restrict__ Z,
                                                            double* __restrict__ gram, double* __restrict__ dblk) {
  const int h = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (h >= d1) return;
  const float* z = Z + (int64_t)h * m;
  double v = 0;
  if ((m & 3) == 0) {
    const float4* z4 = reinterpret_cast<const float4*>(z);
    for (int c = lane; c < (m >> 2); c += 64) {
      const float4 x = z4[c];
      v += (double)x.x * (double)x.x + (double)x.y * (double)x.y + (double)x.z * (double)x.z + (double)x.w * (double)x.w;
    }
  } else {
    for (int c = lane; c < m; c += 64) v += (double)z[c] * (double)z[c];
  }
  v = wave_sum(v);
  if (lane == 0) { gram[h] = v; dblk[h] = (double)N[(int64_t)h * d1 + h]; }
}

// Groups of more than one row: Z_h -= P1_h rZ1 + P2_h rZ2 (P1 == nullptr: left as it is; single: the first term only) and the
// columns' share of gram[h] = Z_h Z_h^T, one pass over Z.  Workgroup = (group, chunk of columns); a wave takes 32 columns at
// a time: the update on v_mfma_f32_16x16x4_f32 (float32 products and sums, as the elements are stored), the new values
// through LDS into operand order, their products on v_mfma_f64_16x16x4_f64.  The waves' sums are added in order and left in
// part[h][chunk][lower tile][256]; score_kernel adds the chunks in order.  Bound by the float32 matrix cores and Z's two
// passes of memory about equally; as a row x 256 columns of scalar products and a second pass for the Grams a swap of two
// groups of 64 rows, 4096 columns took 0.42 + 0.20 ms.  Loads are made from clamped places and dropped where they lie outside: under
// a condition each was waited for by itself, and the launch of both updates took 120 us there instead of 104.
constexpr int GU_LD = 36;
// ROWS rows of a panel (q floats each, contiguous) into S[r * ks + k0 + c], c < kq, zeros past q and past the first `rows` rows;
// by 256 threads, 256 / ROWS of them to a row, four floats at a time where the rows allow it
template <int ROWS>
__device__ __forceinline__ void stage_panel(float* S, int ks, int k0, int kq, const float* __restrict__ P, int q, int rows) {
  constexpr int TPR = 256 / ROWS;
  const int r = threadIdx.x / TPR, l = threadIdx.x % TPR;
  if (r >= ROWS) return;
  float* dst = S + r * ks + k0;
  const bool live = r < rows;
  const float* src = P + (int64_t)(live ? r : rows - 1) * q;      // (a load under a condition is waited for where the branch ends)
  if ((q & 3) == 0 && (reinterpret_cast<uintptr_t>(P) & 15) == 0) {
#pragma unroll 4
    for (int c = 4 * l; c < kq; c += 4 * TPR) {
      const float4 v = *reinterpret_cast<const float4*>(src + c);
      *reinterpret_cast<float4*>(dst + c) = float4{live ? v.x : 0.f, live ? v.y : 0.f, live ? v.z : 0.f, live ? v.w : 0.f};
    }
  } else {
#pragma unroll 4
    for (int c = l; c < kq; c += TPR) {
      const float v = src[min(c, q - 1)];
      dst[c] = (live & (c < q)) ? v : 0.f;
    }
  }
}
template <int RT> struct GroupUpdLds { float zt[4][16 * RT][GU_LD]; };
static __host__ __device__ inline int gu_kq(int q) { return (q + 3) / 4 * 4; }
// The groups of a move's own pivots (g, j; -1: none) take their new rows instead: Z''_g = M1 rZ2 - rZ1 in float64, Z''_j = rZ2.
template <int RT>
__device__ __forceinline__ void group_update(float* gu_lds, TabDims d, float* __restrict__ Z, const float* __restrict__ P1,
                                             const float* __restrict__ P2, const float* __restrict__ rZ1, const float* __restrict__ rZ2,
                                             const double* __restrict__ M1, int single, double* __restrict__ part, int chunk_cols, int chunks,
                                             int g, int j, int h, int chunk) {
  constexpr int NT = RT * (RT + 1) / 2;
  float (*zt)[16 * RT][GU_LD] = reinterpret_cast<float (*)[16 * RT][GU_LD]>(gu_lds);
  float* Ps = gu_lds + 4 * 16 * RT * GU_LD;               // [16 RT][ks]: the rows' coefficients, both pivots' halves side by side
  const int q = d.q, m = d.m, kq = gu_kq(q), K = (P1 && h != g && h != j) ? (single ? kq : 2 * kq) : 0, ks = 2 * kq + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  float* Zh = Z + (int64_t)h * q * m;
  const int c_end = min(m, (chunk + 1) * chunk_cols);
  if (h == g || h == j) {
    for (int col = chunk * chunk_cols + wave * 16 + lc; col - lc < c_end; col += 64)
      for (int i0 = 0; i0 < q; i0 += 16) {
        swd4 acc = {0.0, 0.0, 0.0, 0.0};
        if (h == g && !single) {
          const double* Mi = M1 + min(i0 + lc, q - 1) * q;
          const float* rz = rZ2 + min(col, m - 1);
#pragma unroll 8
          for (int k0 = 0; k0 < q; k0 += 4) {
            const int k = k0 + lr, kc = min(k, q - 1);
            const double at = Mi[kc];
            const float bt = rz[(int64_t)kc * m];
            const double av = k < q ? at : 0.0, bv = k < q ? (double)bt : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
          }
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int i = i0 + 4 * r + lr;
          const int64_t o = (int64_t)i * m + col;
          if (i < q && col < m) Zh[o] = h == g ? (float)(acc[r] - (double)rZ1[o]) : rZ2[o];
        }
      }
  } else if (K) {
    stage_panel<16 * RT>(Ps, ks, 0, kq, P1 + (int64_t)h * q * q, q, q);
    if (!single) stage_panel<16 * RT>(Ps, ks, kq, kq, P2 + (int64_t)h * q * q, q, q);
  }
  __syncthreads();
  swd4 gr[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) gr[t] = swd4{0.0, 0.0, 0.0, 0.0};
  for (int c0 = chunk * chunk_cols + wave * 32; c0 < c_end; c0 += 128) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    f4v acc[RT][2];
    float z[RT][2][4];
#pragma unroll
    for (int t = 0; t < RT; t++)
#pragma unroll
      for (int j = 0; j < 2; j++) {
        acc[t][j] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; r++) {                     // C layout: row 4 (lane / 16) + r, column lane % 16
          const int row = t * 16 + 4 * lr + r, col = c0 + j * 16 + lc;
          z[t][j][r] = Zh[(int64_t)min(row, q - 1) * m + min(col, m - 1)];
        }
      }
    for (int half = 0; half * kq < K; half++) {
      const float* rz = half ? rZ2 : rZ1;
      const float* b0 = rz + min(c0 + lc, m - 1);
      const float* b1 = rz + min(c0 + 16 + lc, m - 1);
      const float* ap = Ps + lc * ks + half * kq + lr;
#pragma unroll 8
      for (int kk = 0; kk < kq; kk += 4) {                  // past q the coefficients are zeros
        const int64_t o = (int64_t)min(kk + lr, q - 1) * m;
        const float b[2] = {b0[o], b1[o]};
#pragma unroll
        for (int t = 0; t < RT; t++) {
          const float av = ap[t * 16 * ks + kk];
#pragma unroll
          for (int j = 0; j < 2; j++) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b[j], acc[t][j], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < RT; t++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int row = t * 16 + 4 * lr + r, col = c0 + j * 16 + lc;
          const bool inside = (row < q) & (col < m);
          const float v = inside ? z[t][j][r] - acc[t][j][r] : 0.f;
          if (K && inside) Zh[(int64_t)row * m + col] = v;
          zt[wave][row][j * 16 + lc] = v;
        }
    // the wave's own part of LDS: in order, no barrier
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s4 = 0; s4 < 8; s4++) {
      double v[RT];
#pragma unroll
      for (int t = 0; t < RT; t++) v[t] = (double)zt[wave][t * 16 + lc][4 * s4 + lr];
#pragma unroll
      for (int t = 0, n = 0; t < RT; t++)
#pragma unroll
        for (int u = 0; u <= t; u++, n++) gr[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t], v[u], gr[n], 0, 0, 0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
  double* red = reinterpret_cast<double*>(gu_lds);        // [NT][256], over zt
  for (int w = 0; w < 4; w++) {
    __syncthreads();
    if (wave == w) {
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          double* p = red + t * 256 + r * 64 + lane;
          *p = w ? *p + gr[t][r] : gr[t][r];
        }
    }
  }
  __syncthreads();
  double* out = part + ((int64_t)h * chunks + chunk) * (NT * 256);
  for (int idx = tid; idx < NT * 256; idx += 256) out[idx] = red[idx];
}
template <int RT>
constexpr size_t group_update_lds(int kq) { return (size_t)(4 * 16 * RT * GU_LD + 16 * RT * (2 * kq + 4)) * 4; }
// the groups' Grams of Z as it stands
template <int RT>
__global__ __launch_bounds__(256, 2) void group_gram_kernel(TabDims d, float* __restrict__ Z, double* __restrict__ part, int chunk_cols) {
  extern __shared__ float gu_lds[];
  group_update<RT>(gu_lds, d, Z, nullptr, nullptr, nullptr, nullptr, nullptr, 0, part, chunk_cols, gridDim.y, -1, -1, blockIdx.x, blockIdx.y);
}
// columns per chunk of the pass over Z: about 1024 workgroups, whole steps of 128 columns
static int gu_chunk_cols(int p, int m) {
  const int chunks = std::max(1, std::min(1024 / std::max(p, 1), (m + 127) / 128));
  return ((m + chunks - 1) / chunks + 127) / 128 * 128;
}
size_t group_part_doubles(int64_t p, int64_t q, int64_t m) {
  if (q <= 1) return 0;
  const int64_t rt = (q + 15) / 16, cc = gu_chunk_cols((int)p, (int)m);
  return (size_t)(p * ((m + cc - 1) / cc) * (rt * (rt + 1) / 2) * 256);
}
static hipError_t launch_group_gram(const TabDims& d, const TabPtrs& t, hipStream_t s) {
  const int cc = gu_chunk_cols(d.p, d.m);
  OSSCAR_BY_TILES(d.q, {
    const size_t lds = group_update_lds<RT>(gu_kq(d.q));
    static_assert(sizeof(GroupUpdLds<RT>) >= RT * (RT + 1) / 2 * 256 * 8, "the reduction shares the tiles' memory");
    if (lds > 65536) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(group_gram_kernel<RT>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(group_gram_kernel<RT>, dim3(d.p, (d.m + cc - 1) / cc), dim3(256), lds, s, d, t.Z, t.part, cc);
  })
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void dblk_copy_kernel(TabDims d, const float* __restrict__ N, double* __restrict__ dblk) {
  const int h = blockIdx.x, q = d.q;
  for (int idx = threadIdx.x; idx < q * q; idx += 256) {
    int r = idx / q, c = idx % q;
    dblk[(int64_t)h * q * q + idx] = (double)nsym(N, d.d1, h * q + r, h * q + c);
  }
}

// The exact change of the objective and whether the pair is taken, from the partial sums of the column phase: lane l adds the
// sums l, l + 64, ... in that order; then the fixed tree of the wave sum.  Known to every lane of every wave that calls it.
__device__ __forceinline__ bool pair_taken(const SearchCtrl* ctrl, int always_accept, const double* __restrict__ dpart, int nparts, double& delta) {
  double dsum = 0;
#pragma unroll 4
  for (int b = threadIdx.x & 63; b < nparts; b += 64) dsum += dpart[b];
  delta = __shfl(wave_sum(dsum), 0);
  return ctrl->notpd == 0 && (always_accept || delta < -ctrl->rel_tol * ctrl->obj);
}
// the outcome of a move, into ctrl and the trace (one thread)
struct PairTrace { int32_t* out = nullptr; int32_t* in = nullptr; float* gap = nullptr; double* obj = nullptr; };
__device__ __forceinline__ void pair_commit(SearchCtrl* ctrl, bool ok, double delta, const int32_t* single, const PairTrace& tr) {
  ctrl->delta = delta;
  const int it = ctrl->iters;
  ctrl->iters = it + 1;
  if (single) { ctrl->g_out = *single; ctrl->g_in = -1; }
  if (ok) { ctrl->obj += delta; ctrl->accepted += 1; } else { ctrl->done = 1; }
  if (tr.out) tr.out[it] = ctrl->g_out;
  if (tr.in) tr.in[it] = ctrl->g_in;
  if (tr.gap) { tr.gap[2 * it] = (float)ctrl->gap_rem; tr.gap[2 * it + 1] = (float)ctrl->gap_add; }
  if (tr.obj) tr.obj[it] = ctrl->obj;
}
// score[h] = Tr(gram_h (sigma dblk_h)^-1), sigma = -1 for kept groups (N_hh = -P_hh), +1 otherwise; one workgroup per group.
// After a move (P1): nothing if it was turned down, and the first workgroup records it (pair_commit) where no other reads it.
// Before the scores, if given: gram_h = the sum of its column chunks (part), and the float64 diagonal block of a group outside the
// pivots takes -= P1D_h P1_h^T + P2D_h P2_h^T (P1; single: the first term only).
template <int RT>
__global__ __launch_bounds__(256) void score_kernel(TabDims d, const int32_t* __restrict__ kept, double* gram, double* dblk,
                                                     double* __restrict__ score, SearchCtrl* ctrl, int skip_if_done,
                                                     const double* __restrict__ part, int chunks, const float* __restrict__ P1,
                                                     const float* __restrict__ P2, const float* __restrict__ P1D,
                                                     const float* __restrict__ P2D, const int32_t* __restrict__ single, PairTrace tr) {
  __shared__ InvLds<RT> L;
  __shared__ double red[4];
  if (skip_if_done && ctrl->done) return;          // a search iteration that changed nothing
  if (P1) {
    const bool ok = ctrl->taken != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) pair_commit(ctrl, ok, ctrl->delta, single, tr);
    if (!ok) return;
  }
  constexpr int NT = RT * (RT + 1) / 2;
  const int h = blockIdx.x, q = d.q, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  double* gram_h = gram + (int64_t)h * q * q;
  double* dblk_h = dblk + (int64_t)h * q * q;
  if (part) {
    const double* ph = part + (int64_t)h * chunks * (NT * 256);
    double sum[NT];
#pragma unroll
    for (int n = 0; n < NT; n++) sum[n] = 0;
    for (int ch = 0; ch < chunks; ch += 4) {              // four chunks of every tile in flight, added in order
      double v[4][NT];
#pragma unroll
      for (int u = 0; u < 4; u++)
#pragma unroll
        for (int n = 0; n < NT; n++) v[u][n] = ph[(int64_t)min(ch + u, chunks - 1) * (NT * 256) + n * 256 + tid];
#pragma unroll
      for (int u = 0; u < 4; u++)
#pragma unroll
        for (int n = 0; n < NT; n++) sum[n] = ch + u < chunks ? sum[n] + v[u][n] : sum[n];
    }
#pragma unroll
    for (int n = 0; n < NT; n++) {
      const double v = sum[n];
      int t = n, br = 0;
      while (t > br) { t -= br + 1; br++; }
      const int r = br * 16 + (tid >> 4), c = t * 16 + (tid & 15);
      if (r < q && c < q) {
        gram_h[r * q + c] = v;
        if (br != t) gram_h[c * q + r] = v;
      }
    }
  }
  if (P1) {
    const int g = single ? *single : ctrl->g_out, j = single ? g : ctrl->g_in;
    if (h != g && h != j) {                       // pivot groups get their blocks in pair_fix_rows
      const int64_t base = (int64_t)h * q * q;
      for (int t = wave; t < NT; t += 4) {
        int br = 0, bc = t;
        while (bc > br) { bc -= br + 1; br++; }
        const int i = br * 16 + lc, l = bc * 16 + lc;
        swd4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int half = 0; half < (single ? 1 : 2); half++) {
          const float* A = half ? P2D : P1D;
          const float* B = half ? P2 : P1;
          const float* Ai = A + base + min(i, q - 1) * q;
          const float* Bl = B + base + min(l, q - 1) * q;
#pragma unroll 8
          for (int k0 = 0; k0 < q; k0 += 4) {
            const int k = k0 + lr, kc = min(k, q - 1);
            const float at = Ai[kc], bt = Bl[kc];
            const double av = k < q ? (double)at : 0.0, bv = k < q ? (double)bt : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
          }
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int a = br * 16 + 4 * r + lr, b = bc * 16 + lc;
          if (a < q && b <= a) {
            const double v = dblk_h[a * q + b] - acc[r];
            dblk_h[a * q + b] = v; dblk_h[b * q + a] = v;
          }
        }
      }
    }
  }
  __syncthreads();
  const double sigma = kept[h] ? -1.0 : 1.0;
  double contrib = 0;
  const bool bad = inv_sym<4, (NT + 3) / 4, RT>(q, L, [&](int i, int j) { return sigma * dblk_h[i * q + j]; },
                                                [&](int i, int j, double v) { contrib += (i == j ? 1.0 : 2.0) * v * gram_h[i * q + j]; });
  contrib = wave_sum(contrib);
  if (lane == 0) red[wave] = contrib;
  if (bad && lane == 0) ctrl->notpd = 1;
  __syncthreads();
  if (tid == 0) score[h] = red[0] + red[1] + red[2] + red[3];
}
// groups of one row: one thread per group
__global__ __launch_bounds__(256) void score_q1_kernel(int p, const int32_t* __restrict__ kept, const double* __restrict__ gram,
                                                        const double* __restrict__ dblk, double* __restrict__ score,
                                                        SearchCtrl* ctrl, int skip_if_done) {
  if (skip_if_done && ctrl->done) return;
  const int h = blockIdx.x * 256 + threadIdx.x;
  if (h >= p) return;
  double a = (kept[h] ? -1.0 : 1.0) * dblk[h];
  if (!(a > 0.0)) { ctrl->notpd = 1; a = 1.0; }
  score[h] = gram[h] / a;
}
struct ScoreUpdate { const double* part = nullptr; const float *P1 = nullptr, *P2 = nullptr, *P1D = nullptr, *P2D = nullptr; const int32_t* single = nullptr; PairTrace trace; };
static void launch_score(const TabDims& d, const int32_t* kept, double* gram, double* dblk, double* score, SearchCtrl* ctrl, int skip_if_done,
                         hipStream_t s, const ScoreUpdate& u = ScoreUpdate()) {
  if (d.q == 1) {
    hipLaunchKernelGGL(score_q1_kernel, dim3((d.p + 255) / 256), dim3(256), 0, s, d.p, kept, gram, dblk, score, ctrl, skip_if_done);
    return;
  }
  const int cc = gu_chunk_cols(d.p, d.m);
  OSSCAR_BY_TILES(d.q, hipLaunchKernelGGL(score_kernel<RT>, dim3(d.p), dim3(256), 0, s, d, kept, gram, dblk, score, ctrl, skip_if_done, u.part,
                                          (d.m + cc - 1) / cc, u.P1, u.P2, u.P1D, u.P2D, u.single, u.trace))
}

// the two halves of the refresh: the per-group Gram blocks and diagonal blocks (one pass over Z and the diagonal of N),
// then the scores from them; a caller may run the first half on another stream
static hipError_t launch_refresh_blocks(const TabDims& d, const TabPtrs& t, hipStream_t s) {
  if (d.q == 1) {
    hipLaunchKernelGGL(gram_dblk_q1_kernel, dim3((d.d1 + 3) / 4), dim3(256), 0, s, d.d1, d.m, t.N, t.Z, t.gram, t.dblk);
  } else {
    const hipError_t e = launch_group_gram(d, t, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(dblk_copy_kernel, dim3(d.p), dim3(256), 0, s, d, t.N, t.dblk);
  }
  return hipGetLastError();
}
hipError_t launch_refresh_scores(const TabDims& d, const TabPtrs& t, hipStream_t s) {
  const hipError_t e = launch_refresh_blocks(d, t, s);
  if (e != hipSuccess) return e;
  ScoreUpdate u;
  u.part = t.part;
  launch_score(d, t.kept, t.gram, t.dblk, t.score, t.ctrl, 0, s, u);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// one search iteration
// ------------------------------------------------------------------------------------------------
// argmin of the removal costs over kept groups, argmax of the addition gains over the others (lowest
// index on ties), and the relative gap to the second best of each.
// the best value (smallest), the next one, and the index of the best, the lowest of equal ones; -1: none
struct TwoBest {
  double v1, v2;
  int i;
  __device__ __forceinline__ void clear() { v1 = v2 = INFINITY; i = -1; }
  __device__ __forceinline__ void take(double v, int h) {          // ascending h: a strict comparison keeps the lowest index
    const bool lt = v < v1;
    v2 = lt ? v1 : fmin(v2, v);
    v1 = lt ? v : v1; i = lt ? h : i;
  }
  __device__ __forceinline__ void join(const TwoBest& b) {
    const bool t = (b.i >= 0) & ((i < 0) | (b.v1 < v1) | ((b.v1 == v1) & (b.i < i)));
    v2 = fmin(fmin(v2, b.v2), t ? v1 : b.v1);
    v1 = t ? b.v1 : v1; i = t ? b.i : i;
  }
  // the best of the wave, in every lane
  __device__ __forceinline__ void over_wave() {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      TwoBest b;
      b.v1 = __shfl_xor(v1, o); b.v2 = __shfl_xor(v2, o); b.i = __shfl_xor(i, o);
      join(b);
    }
  }
  __device__ __forceinline__ double gap() const { return isfinite(v2) ? fabs(v2 - v1) / fmax(fabs(v1), 1e-300) : INFINITY; }
};
// Leaving group (of the kept ones: the smallest score) and entering group (of the others: the largest, held negated), known to
// every thread of a workgroup of T.  In steps of a wave and one exchange through LDS: as a tree over 1024 threads in LDS the
// selection was a launch of 4.1 us at 256 groups.
template <int T>
__device__ __forceinline__ void pick_pair(int p, const int32_t* __restrict__ kept, const double* __restrict__ score, TwoBest& out, TwoBest& in) {
  __shared__ TwoBest s_out[T / 64], s_in[T / 64];
  const int tid = threadIdx.x;
  out.clear(); in.clear();
#pragma unroll 4
  for (int h = tid; h < p; h += T) {
    const double v = score[h];
    const bool k = kept[h] != 0;
    out.take(k ? v : INFINITY, h);
    in.take(k ? INFINITY : -v, h);
  }
  out.over_wave(); in.over_wave();
  if ((tid & 63) == 0) { s_out[tid >> 6] = out; s_in[tid >> 6] = in; }
  __syncthreads();
  out = s_out[0]; in = s_in[0];
#pragma unroll 3
  for (int w = 1; w < T / 64; w++) { out.join(s_out[w]); in.join(s_in[w]); }
}
// the pair a move takes: the picked one, or the one the caller names; false (of every thread alike): there is none.
// record: this thread writes it to ctrl
__device__ __forceinline__ bool settle_pair(const TwoBest& out, const TwoBest& in, int forced_out, int forced_in, const int32_t* __restrict__ kept,
                                            SearchCtrl* ctrl, bool record, int& g, int& j) {
  g = forced_out >= 0 ? forced_out : out.i; j = forced_out >= 0 ? forced_in : in.i;
  if (g < 0 || j < 0 || (forced_out >= 0 && (!kept[g] || kept[j]))) {
    if (record) { ctrl->done = 1; ctrl->g_out = -1; ctrl->g_in = -1; }
    return false;
  }
  if (record) { ctrl->g_out = g; ctrl->g_in = j; ctrl->gap_rem = out.gap(); ctrl->gap_add = in.gap(); }
  return true;
}
__global__ __launch_bounds__(1024) void select_kernel(TabDims d, const int32_t* __restrict__ kept,
                                                       const double* __restrict__ score, SearchCtrl* ctrl, int forced_out,
                                                       int forced_in) {
  if (ctrl->done || ctrl->pause) return;
  TwoBest out, in;
  pick_pair<1024>(d.p, kept, score, out, in);
  int g, j;
  settle_pair(out, in, forced_out, forced_in, kept, ctrl, threadIdx.x == 0, g, j);
}

// ------------------------------------------------------------------------------------------------
// Exact entering rule: with the leaving group g fixed, every candidate j is scored at the state WITHOUT g (Case 1 of
// Proposition 4.1 applied to the blocks the score needs, then eq. (impact) there), i.e. by the exact gain of the pair.
// Sweeping g out changes   N_jj -> N_jj - Y N_gj,   Z_j -> Z_j - Y Z_g,   Y = N_jg N_gg^-1,
// so with C_j = Z_j Z_g^T (exact_cross_kernel) the Gram of the new rows is
//   M_j = Z_j Z_j^T - Y C_j^T - C_j Y^T + Y (Z_g Z_g^T) Y^T          and the score is Tr(S'_j^-1 M_j).
// ------------------------------------------------------------------------------------------------
// cross[i][c] = <Z_i, Z_{g, c}> for every row i; one wave per row, Zg = the copy of the rows of g (q x m)
__global__ __launch_bounds__(256) void exact_cross_kernel(TabDims d, const float* __restrict__ Z, const float* __restrict__ Zg,
                                                           const SearchCtrl* __restrict__ ctrl, double* __restrict__ cross) {
  if (ctrl->done) return;
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= d.d1) return;
  const float* zi = Z + (int64_t)row * d.m;
  for (int c = 0; c < d.q; c++) {
    const float* zg = Zg + (int64_t)c * d.m;
    double v = 0;
    for (int col = lane; col < d.m; col += 64) v += (double)zi[col] * (double)zg[col];
    v = wave_sum(v);
    if (lane == 0) cross[(int64_t)row * d.q + c] = v;
  }
}

// groups of one row: the score itself, one thread per group
__global__ __launch_bounds__(256) void exact_q1_kernel(TabDims d, const float* __restrict__ C1, const double* __restrict__ cross,
                                                        const double* __restrict__ gram, const double* __restrict__ dblk,
                                                        const int32_t* __restrict__ kept, SearchCtrl* ctrl,
                                                        double* __restrict__ xscore) {
  if (ctrl->done) return;
  const int h = blockIdx.x * 256 + threadIdx.x;
  if (h >= d.p) return;
  if (kept[h]) { xscore[h] = 0.0; return; }
  const int g = ctrl->g_out;
  const double x = (double)C1[h], y = x / dblk[g];
  double sp = dblk[h] - y * x;
  const double mj = gram[h] - 2.0 * y * cross[h] + y * y * gram[g];
  if (!(sp > 0.0)) { ctrl->notpd = 1; sp = 1.0; }
  xscore[h] = mj / sp;
}

// groups of q rows: the blocks S'_j -> xdblk[j], M_j -> xgram[j] (kept groups: -I and 0, which score_kernel turns into 0)
__global__ __launch_bounds__(256) void exact_blocks_kernel(TabDims d, const float* __restrict__ C1, const double* __restrict__ cross,
                                                            const double* __restrict__ gram, const double* __restrict__ dblk,
                                                            const int32_t* __restrict__ kept, SearchCtrl* ctrl,
                                                            double* __restrict__ xgram, double* __restrict__ xdblk) {
  extern __shared__ double xsh[];      // Dg (later T = Y Gg), X, Y: q*q each; then 256 doubles for the inverse
  __shared__ int32_t bad;
  if (ctrl->done) return;
  const int q = d.q, qq = q * q, tid = threadIdx.x, j = blockIdx.x, g = ctrl->g_out, j0 = j * q;
  double* outS = xdblk + (int64_t)j * qq;
  double* outM = xgram + (int64_t)j * qq;
  if (kept[j]) {
    for (int idx = tid; idx < qq; idx += 256) { outS[idx] = (idx / q == idx % q) ? -1.0 : 0.0; outM[idx] = 0.0; }
    return;
  }
  double* Dg = xsh; double* X = xsh + qq; double* Y = xsh + 2 * qq; double* buf = xsh + 3 * qq;
  if (tid == 0) bad = 0;
  for (int idx = tid; idx < qq; idx += 256) {
    Dg[idx] = dblk[(int64_t)g * qq + idx];                                   // N_gg, negative definite
    X[idx] = (double)C1[(int64_t)(j0 + idx / q) * q + idx % q];              // N(j_r, g_c)
  }
  small_inverse<4>(Dg, q, -1, &bad, buf);
  for (int idx = tid; idx < qq; idx += 256) {                                // Y = X Dg
    const int r = idx / q, c = idx % q;
    double v = 0;
    for (int k = 0; k < q; k++) v += X[r * q + k] * Dg[k * q + c];
    Y[idx] = v;
  }
  __syncthreads();
  const double* Gg = gram + (int64_t)g * qq;
  const double* Gj = gram + (int64_t)j * qq;
  const double* Sj = dblk + (int64_t)j * qq;
  const double* Cj = cross + (int64_t)j0 * q;                               // C_j[r][c] = <Z_{j,r}, Z_{g,c}>
  double* Tm = Dg;                                                           // T = Y Gg overwrites Dg
  for (int idx = tid; idx < qq; idx += 256) {
    const int r = idx / q, c = idx % q;
    double sv = 0;
    for (int k = 0; k < q; k++) sv += Y[r * q + k] * X[c * q + k];
    outS[idx] = Sj[idx] - sv;                                                // S' = N_jj - Y N_gj
  }
  __syncthreads();
  for (int idx = tid; idx < qq; idx += 256) {
    const int r = idx / q, c = idx % q;
    double v = 0;
    for (int k = 0; k < q; k++) v += Y[r * q + k] * Gg[k * q + c];
    Tm[idx] = v;
  }
  __syncthreads();
  for (int idx = tid; idx < qq; idx += 256) {
    const int r = idx / q, c = idx % q;
    double v = Gj[idx];
    for (int k = 0; k < q; k++) v += -Y[r * q + k] * Cj[c * q + k] - Cj[r * q + k] * Y[c * q + k] + Tm[r * q + k] * Y[c * q + k];
    outM[idx] = v;
  }
  if (tid == 0 && bad) ctrl->notpd = 1;
}

// entering group = argmax of the exact scores over the groups outside the kept set (lowest index on ties)
__global__ __launch_bounds__(1024) void select_in_kernel(TabDims d, const int32_t* __restrict__ kept,
                                                          const double* __restrict__ xscore, SearchCtrl* ctrl) {
  if (ctrl->done) return;
  TwoBest out, in;
  pick_pair<1024>(d.p, kept, xscore, out, in);
  if (threadIdx.x != 0) return;
  if (in.i < 0) { ctrl->done = 1; ctrl->g_out = -1; ctrl->g_in = -1; return; }
  ctrl->g_in = in.i;
  ctrl->gap_add = in.gap();
}

// Opening of a move: the selection, the panels of both pivots (C1, C2; 64 rows per workgroup, through LDS where the pivot rows
// of N hold them), copies of their Z rows, and the q x q algebra.  Nothing here waits for anything but the selection, which
// every workgroup makes for itself (`pick`; otherwise ctrl holds the pair).  single != nullptr: removal of the one group
// *single, no second pivot.  Workgroups: with `algebra` the first one makes the q x q matrices straight from N; then
// `row_blocks` each for C1, C2 and the two copies.
// small layout (doubles, each q*q): [0] Dg, [1] Njg, [2] M1 = Dg Ngj, [3] Dj' , [4] W2Dj = -M1 Dj'; single: Dg only (the
// others are written as zeros for one-row groups, whose bulk kernels always take both terms).
// Bound by the algebra's two chains of q pivots; the panels run beside it.  As three launches (selection, panels, algebra) the
// same work took 4.1 + 3.5 + 9.8 us at 256 groups of 9 rows, as one 11.3 us.
// PICK_MOST: every workgroup reads all scores; past 8 per thread a launch of its own makes the selection.
constexpr int PICK_MOST = 2048;
template <int RT>
__global__ __launch_bounds__(256) void pair_open_kernel(TabDims d, const float* __restrict__ N, const float* __restrict__ Z,
                                                         const int32_t* __restrict__ kept, const double* __restrict__ score, SearchCtrl* ctrl,
                                                         float* __restrict__ C1, float* __restrict__ C2, float* __restrict__ Zg,
                                                         float* __restrict__ Zj, double* __restrict__ small, const int32_t* __restrict__ single,
                                                         int pick, int forced_out, int forced_in, int algebra, int row_blocks) {
  extern __shared__ double psm[];      // three q x q matrices with rows of q + 1 and one of floats, or 64 x 65 floats
  __shared__ InvLds<RT> L;
  if (ctrl->done) return;
  const int q = d.q, tid = threadIdx.x;
  int g, j;
  if (single) g = j = *single;
  else if (pick) {
    TwoBest out, in;
    pick_pair<256>(d.p, kept, score, out, in);
    if (!settle_pair(out, in, forced_out, forced_in, kept, ctrl, blockIdx.x == 0 && tid == 0, g, j)) return;
  } else { g = ctrl->g_out; j = ctrl->g_in; }
  const int64_t ld = d.d1;
  const int b = (int)blockIdx.x - algebra;
  if (b >= 0) {
    const int part = b / row_blocks, x = b % row_blocks, second = part & 1, t0 = (second ? j : g) * q;
    if (part >= 2) {
      const float* src = Z + (int64_t)t0 * d.m;
      float* dst = second ? Zj : Zg;
      for (int64_t idx = x * 256 + tid; idx < (int64_t)q * d.m; idx += (int64_t)row_blocks * 256) dst[idx] = src[idx];
      return;
    }
    float (*T)[65] = reinterpret_cast<float (*)[65]>(psm);
    float* C = second ? C2 : C1;
    const int i0 = x * 64, ni = min(64, d.d1 - i0);
    if (i0 + ni <= t0) {                                   // above the pivot: the pivot's rows of N, along i
      for (int idx = tid; idx < 64 * q; idx += 256) {
        const int c = idx >> 6, r = idx & 63;
        if (r < ni) T[r][c] = N[(int64_t)(t0 + c) * ld + i0 + r];
      }
      __syncthreads();
      for (int idx = tid; idx < ni * q; idx += 256) C[(int64_t)i0 * q + idx] = T[idx / q][idx % q];
      return;
    }
    for (int idx = tid; idx < ni * q; idx += 256) C[(int64_t)i0 * q + idx] = nsym(N, ld, i0 + idx / q, t0 + idx % q);
    return;
  }
  constexpr int T = (RT * (RT + 1) / 2 + 3) / 4;
  const int qq = q * q, qs = q + 1, g0 = g * q, j0 = j * q;
  double* Dg = small; double* Njg = small + qq; double* M1 = small + 2 * qq; double* Dj = small + 3 * qq;
  double* W2Dj = small + 4 * qq;
  double* X0 = psm; double* X1 = psm + q * qs; double* X2 = psm + 2 * q * qs;
  float* X3 = reinterpret_cast<float*>(psm + 3 * q * qs);       // N_jj
  if (!single) {
#pragma unroll 4
    for (int idx = tid; idx < qq; idx += 256) {
      const int r = idx / q, c = idx % q;
      const float ngj = nsym(N, ld, j0 + r, g0 + c), njj = nsym(N, ld, j0 + r, j0 + c);
      Njg[idx] = (double)ngj;                                   // N(j_r, g_c)
      X1[r * qs + c] = (double)ngj;
      X3[r * qs + c] = njj;
    }
  }
  // kept pivot: N_gg = -P_gg is negative definite
  bool bad = inv_sym<4, T, RT>(q, L, [&](int r, int c) { return -(double)nsym(N, ld, g0 + r, g0 + c); },
                               [&](int r, int c, double v) { X0[r * qs + c] = X0[c * qs + r] = -v; Dg[r * q + c] = Dg[c * q + r] = -v; });
  __syncthreads();
  if (single) {
    // Case 1 alone: with M1 = 0 and Dj' = 0 every term of the second sweep vanishes
    if (q == 1 && tid == 0) { M1[0] = 0.0; Dj[0] = 0.0; W2Dj[0] = 0.0; Njg[0] = 0.0; }
  } else {
    mm_small<RT>(q, [&](int i, int k) { return X0[i * qs + k]; }, [&](int k, int c) { return X1[c * qs + k]; },      // M1 = Dg Ngj
                 [&](int i, int c, double v) { X2[i * qs + c] = v; M1[i * q + c] = v; });
    __syncthreads();
    mm_small<RT>(q, [&](int i, int k) { return X1[i * qs + k]; }, [&](int k, int c) { return X2[k * qs + c]; },      // N'_jj = N_jj - N_jg M1
                 [&](int i, int c, double v) { X0[i * qs + c] = (double)X3[i * qs + c] - v; });
    __syncthreads();
    // entering pivot: Schur complement, positive definite
    bad |= inv_sym<4, T, RT>(q, L, [&](int r, int c) { return X0[r * qs + c]; },
                             [&](int r, int c, double v) { X1[r * qs + c] = X1[c * qs + r] = v; Dj[r * q + c] = Dj[c * q + r] = v; });
    __syncthreads();
    mm_small<RT>(q, [&](int i, int k) { return -X2[i * qs + k]; }, [&](int k, int c) { return X1[k * qs + c]; },     // W2Dj, W2 = N'_gj = -M1
                 [&](int i, int c, double v) { W2Dj[i * q + c] = v; });
  }
  if (bad && (tid & 63) == 0) ctrl->notpd = 1;
}

// Column phase of the pair: rZ1 = Dg Zg ; Z'j = Zj - Njg rZ1 ; rZ2 = Dj' Z'j (both written in place of Zg, Zj) and
// delta = -<Zg, rZ1> - <Z'j, rZ2>, one partial sum per workgroup in dpart (added up in a fixed order by the acceptance
// test, so that the result does not depend on scheduling).  16 columns per workgroup, a wave = 16 rows, float64 matrix cores;
// the q x q matrices come from L2 (a row's 4 k are 32 bytes).
constexpr int PC_COLS = 16;
template <int RT>
__device__ __forceinline__ void pair_cols(TabDims d, float* __restrict__ Zg, float* __restrict__ Zj, const double* __restrict__ small,
                                          double* __restrict__ dpart, const int32_t* __restrict__ single, int block) {
  __shared__ double ta[16 * RT][PC_COLS + 1], tb[16 * RT][PC_COLS + 1];
  __shared__ double red[4];
  const int q = d.q, qq = q * q, m = d.m, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const double* Dg = small; const double* Njg = small + qq; const double* Dj = small + 3 * qq;
  const int i0 = wave * 16, col = block * PC_COLS + lc;
  const bool live = col < m, mine = i0 < q;
  const int tcol = block * PC_COLS + (tid & 15);
#pragma unroll
  for (int u = 0; u < RT; u++) {                             // (loads from clamped places: under a condition each is waited for)
    const int r = (tid >> 4) + 16 * u;
    const float v = Zg[(int64_t)min(r, q - 1) * m + min(tcol, m - 1)];
    ta[r][tid & 15] = ((r < q) & (tcol < m)) ? (double)v : 0.0;
  }
  float zj[4];
#pragma unroll
  for (int r = 0; r < 4; r++) zj[r] = single ? 0.f : Zj[(int64_t)min(i0 + 4 * r + lr, q - 1) * m + min(col, m - 1)];
  __syncthreads();
  auto product = [&](const double* A, double (*B)[PC_COLS + 1]) {
    swd4 acc = {0.0, 0.0, 0.0, 0.0};
    if (mine) {
      const double* Ai = A + min(i0 + lc, q - 1) * q;
#pragma unroll 8
      for (int k0 = 0; k0 < q; k0 += 4) {
        const int k = k0 + lr;
        const double at = Ai[min(k, q - 1)], av = k < q ? at : 0.0, bv = k < q ? B[k][lc] : 0.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
      }
    }
    return acc;
  };
  double part = 0;
  swd4 v = product(Dg, ta);                                  // tb = rZ1 = Dg zg
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int i = i0 + 4 * r + lr;
    if (mine && i < q) {
      part -= ta[i][lc] * v[r];
      tb[i][lc] = v[r];
      if (live) Zg[(int64_t)i * m + col] = (float)v[r];
    }
  }
  if (!single) {
    __syncthreads();
    v = product(Njg, tb);                                    // ta = z'j = zj - Njg tb
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = i0 + 4 * r + lr;
      if (mine && i < q) ta[i][lc] = (live ? (double)zj[r] : 0.0) - v[r];
    }
    __syncthreads();
    v = product(Dj, ta);                                     // rZ2 = Dj' z'j
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = i0 + 4 * r + lr;
      if (mine && i < q) {
        part -= ta[i][lc] * v[r];
        if (live) Zj[(int64_t)i * m + col] = (float)v[r];
      }
    }
  } else if (q == 1 && wave == 0 && lr == 0 && live) {
    Zj[col] = 0.f;
  }
  part = wave_sum(part);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (tid == 0) dpart[block] = red[0] + red[1] + red[2] + red[3];
}

// groups of one row: the test in a launch of its own, before the bulk kernels
__global__ __launch_bounds__(64) void pair_accept_kernel(SearchCtrl* ctrl, int always_accept, PairTrace tr, const int32_t* __restrict__ single,
                                                         const double* __restrict__ dpart, int nparts) {
  if (ctrl->done) return;
  double delta;
  const bool ok = pair_taken(ctrl, always_accept, dpart, nparts, delta);
  if (threadIdx.x == 0) pair_commit(ctrl, ok, delta, single, tr);
}

// bulk panels: P1 = C1, P2 = C2 - C1 M1, P1D = P1 Dg, P2D = P2 Dj', with the rows of both pivots zeroed;
// and the new pivot rows of N and Z, the diagonal blocks (float64) and the membership flags.
// 16 rows per workgroup, a wave = 16 columns, float64 matrix cores; the q x q matrices come from L2.  single: P1 and P1D only.
template <int RT>
__device__ __forceinline__ void pair_panels(TabDims d, const float* __restrict__ C1, const float* __restrict__ C2, const double* __restrict__ small,
                                            const SearchCtrl* __restrict__ ctrl, float* __restrict__ P1, float* __restrict__ P2,
                                            float* __restrict__ P1D, float* __restrict__ P2D, const int32_t* __restrict__ single, int block) {
  __shared__ double sc1[16][16 * RT + 1], sc2[16][16 * RT + 1];
  const int q = d.q, qq = q * q, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const int g0 = (single ? *single : ctrl->g_out) * q, j0 = (single ? *single : ctrl->g_in) * q;
  const double* Dg = small; const double* M1 = small + 2 * qq; const double* Dj = small + 3 * qq;
  const int i0 = block * 16, j = wave * 16 + lc, ni = min(16, d.d1 - i0);
#pragma unroll 4
  for (int idx = tid; idx < 16 * q; idx += 256) {
    const float v = C1[(int64_t)i0 * q + min(idx, ni * q - 1)];
    sc1[idx / q][idx % q] = idx < ni * q ? (double)v : 0.0;
  }
  float c2[4];
#pragma unroll
  for (int r = 0; r < 4; r++) c2[r] = single ? 0.f : C2[(int64_t)(i0 + min(4 * r + lr, ni - 1)) * q + min(j, q - 1)];
  __syncthreads();
  auto product = [&](const double (*A)[16 * RT + 1], const double* B) {
    swd4 acc = {0.0, 0.0, 0.0, 0.0};
    const double* Bj = B + min(j, q - 1);
#pragma unroll 8
    for (int k0 = 0; k0 < q; k0 += 4) {
      const int k = k0 + lr;
      const double bt = Bj[min(k, q - 1) * q], av = k < q ? A[lc][k] : 0.0, bv = k < q ? bt : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
    }
    return acc;
  };
  swd4 v1 = {0.0, 0.0, 0.0, 0.0}, v2 = v1;
  const bool mine = wave < RT;
  if (mine) v1 = product(sc1, Dg);
  if (!single) {
    if (mine) {
      const swd4 v = product(sc1, M1);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int i = 4 * r + lr;
        sc2[i][j] = (i < ni && j < q) ? (double)c2[r] - v[r] : 0.0;
      }
    }
    __syncthreads();
    if (mine) v2 = product(sc2, Dj);
  }
  if (!mine || j >= q) return;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int l = 4 * r + lr, i = i0 + l;
    if (l >= ni) continue;
    const bool piv = (i >= g0 && i < g0 + q) || (i >= j0 && i < j0 + q);
    const int64_t o = (int64_t)i * q + j;
    P1[o] = piv ? 0.f : (float)sc1[l][j];
    P1D[o] = piv ? 0.f : (float)v1[r];
    if (!single) { P2[o] = piv ? 0.f : (float)sc2[l][j]; P2D[o] = piv ? 0.f : (float)v2[r]; }
    else if (q == 1) { P2[o] = 0.f; P2D[o] = 0.f; }
  }
}

// Both follow from the q x q matrices alone, so they share a launch (rows of the panels first, then the columns): apart, with
// the acceptance test between them, they took 6.1 + 2.3 + 7.0 us at 256 groups of 9 rows, as one 6.9 us.
template <int RT>
__global__ __launch_bounds__(256) void pair_mid_kernel(TabDims d, const float* __restrict__ C1, const float* __restrict__ C2,
                                                        const double* __restrict__ small, const SearchCtrl* __restrict__ ctrl,
                                                        float* __restrict__ P1, float* __restrict__ P2, float* __restrict__ P1D,
                                                        float* __restrict__ P2D, float* __restrict__ Zg, float* __restrict__ Zj,
                                                        double* __restrict__ dpart, const int32_t* __restrict__ single, int row_blocks) {
  if (ctrl->done) return;
  if ((int)blockIdx.x < row_blocks) pair_panels<RT>(d, C1, C2, small, ctrl, P1, P2, P1D, P2D, single, blockIdx.x);
  else pair_cols<RT>(d, Zg, Zj, small, dpart, single, (int)blockIdx.x - row_blocks);
}

// New pivot rows (after both sweeps), for every l outside the pivots:
//   N''(g_r, l) = -P1D[l][r] - sum_c W2[r][c] P2D[l][c],  W2 = -M1     (= -P1D[l][r] + sum_c M1[r][c] P2D[l][c])
//   N''(j_r, l) =  P2D[l][r]
// pivot-pivot blocks: N''_gg = -Dg - W2 Dj' W2^T, N''_jj = -Dj', N''(g, j) = W2 Dj'.
// Z''_g = -rZ1 + M1 rZ2, Z''_j = rZ2.  Diagonal blocks of the other groups are updated in float64.
// 16 rows l of N per workgroup; the first one also writes the pivot-pivot blocks and the flags.
template <int RT>
__device__ __forceinline__ void pair_fix_rows(TabDims d, float* __restrict__ N, const float* __restrict__ P1D, const float* __restrict__ P2D,
                                              const double* __restrict__ small, double* __restrict__ dblk, int32_t* __restrict__ kept,
                                              const int32_t* __restrict__ single, int g, int j, int block) {
  __shared__ float tg[16][16 * RT + 1], tj[16][16 * RT + 1];
  const int q = d.q, qq = q * q, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15, g0 = g * q, j0 = j * q;
  const double* Dg = small; const double* M1 = small + 2 * qq; const double* Dj = small + 3 * qq; const double* W2Dj = small + 4 * qq;
  const int64_t ld = d.d1;
  const int l0 = block * 16, nl = min(16, d.d1 - l0);
  if (!single) {
#pragma unroll 4
    for (int idx = tid; idx < 16 * q; idx += 256) {
      const float v = P2D[(int64_t)l0 * q + min(idx, nl * q - 1)];
      tj[idx / q][idx % q] = idx < nl * q ? v : 0.f;
    }
    __syncthreads();
  }
  if (wave < RT) {
    const int r0 = wave * 16 + lc;                 // pivot row
    swd4 acc = {0.0, 0.0, 0.0, 0.0};
    if (!single) {
      const double* Mr = M1 + min(r0, q - 1) * q;
#pragma unroll 8
      for (int k0 = 0; k0 < q; k0 += 4) {
        const int k = k0 + lr;
        const double bt = Mr[min(k, q - 1)], av = k < q ? (double)tj[lc][k] : 0.0, bv = k < q ? bt : 0.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int l = 4 * r + lr;
      if (l < nl && r0 < q) tg[l][r0] = (float)(acc[r] - (double)P1D[(int64_t)(l0 + l) * q + r0]);
    }
  }
  __syncthreads();
  auto write = [&](int t0, const float (*T)[16 * RT + 1], int other) {
    auto outside = [&](int l) { return !(l >= t0 && l < t0 + q) && !(l >= other && l < other + q); };
    if (l0 + nl <= t0) {                           // the pivot's rows of N, along l
      for (int idx = tid; idx < 16 * q; idx += 256) {
        const int l = idx & 15, r = idx >> 4;
        if (l < nl && outside(l0 + l)) N[(int64_t)(t0 + r) * ld + l0 + l] = T[l][r];
      }
    } else {
      for (int idx = tid; idx < nl * q; idx += 256) {
        const int l = idx / q, r = idx % q, row = l0 + l, pr = t0 + r;
        if (!outside(row)) continue;
        if (row < pr) N[(int64_t)pr * ld + row] = T[l][r]; else N[(int64_t)row * ld + pr] = T[l][r];
      }
    }
  };
  write(g0, tg, j0);
  if (!single) write(j0, tj, g0);
  if (block != 0) return;
  auto set_gg = [&](int r, int c, double ngg) {    // N''_gg
    dblk[(int64_t)g * qq + r * q + c] = ngg;
    if (c <= r) N[(int64_t)(g0 + r) * ld + g0 + c] = (float)ngg;
  };
  if (single) {
    for (int idx = tid; idx < qq; idx += 256) set_gg(idx / q, idx % q, -Dg[idx]);
  } else {
    // - W2 Dj' W2^T = + (W2 Dj') M1^T
    mm_small<RT>(q, [&](int i, int k) { return W2Dj[i * q + k]; }, [&](int k, int c) { return M1[c * q + k]; },
                 [&](int i, int c, double v) { set_gg(i, c, v - Dg[i * q + c]); });
    for (int idx = tid; idx < qq; idx += 256) {
      const int r = idx / q, c = idx % q;
      const double njj = -Dj[idx], ngj = W2Dj[idx];                            // N''(g_r, j_c)
      dblk[(int64_t)j * qq + idx] = njj;
      if (c <= r) N[(int64_t)(j0 + r) * ld + j0 + c] = (float)njj;
      if (g0 > j0) N[(int64_t)(g0 + r) * ld + j0 + c] = (float)ngj;
      else N[(int64_t)(j0 + c) * ld + g0 + r] = (float)ngj;
    }
  }
  if (tid == 0) { kept[g] = 0; if (!single) kept[j] = 1; }
}
// groups of one row: these rows of N (row_blocks workgroups), then 64 columns of the two rows of Z each
__global__ __launch_bounds__(256) void pair_fix_q1_kernel(TabDims d, float* __restrict__ N, float* __restrict__ Z,
                                                           const float* __restrict__ P1D, const float* __restrict__ P2D,
                                                           const float* __restrict__ rZ1, const float* __restrict__ rZ2,
                                                           const double* __restrict__ small, const SearchCtrl* __restrict__ ctrl,
                                                           double* __restrict__ dblk, int32_t* __restrict__ kept,
                                                           const int32_t* __restrict__ single, int row_blocks) {
  if (ctrl->done) return;
  const int g = single ? *single : ctrl->g_out, j = single ? g : ctrl->g_in, m = d.m;
  if ((int)blockIdx.x < row_blocks) { pair_fix_rows<1>(d, N, P1D, P2D, small, dblk, kept, single, g, j, blockIdx.x); return; }
  const int col = ((int)blockIdx.x - row_blocks) * 64 + (int)threadIdx.x;
  if (threadIdx.x >= 64 || col >= m) return;
  Z[(int64_t)g * m + col] = (float)((single ? 0.0 : small[2] * (double)rZ2[col]) - (double)rZ1[col]);
  if (!single) Z[(int64_t)j * m + col] = rZ2[col];
}

// bulk update of the lower triangle: N[i][l] -= sum_c P1D[i][c] P1[l][c] + P2D[i][c] P2[l][c] (single: the first term only).
// 64 x 64 tiles, four waves x (2 x 2) v_mfma_f32_16x16x4_f32, the panels' rows whole in LDS (rows of 2 kq + 4 floats: the 16
// rows x 4 k of an operand read lie in different banks).  Bound by N's read and write; the requests for N go first.
// The pivots' rows and columns are left to pair_fix_rows (g0, j0: their first rows; single: j0 = g0).
__device__ __forceinline__ void update_N(float* un_lds, TabDims d, float* __restrict__ N, const float* __restrict__ P1,
                                         const float* __restrict__ P2, const float* __restrict__ P1D, const float* __restrict__ P2D,
                                         int single, int g0, int j0, int tile) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  int tr = (int)((sqrtf(8.f * (float)tile + 1.f) - 1.f) * 0.5f);
  while ((int64_t)(tr + 1) * (tr + 2) / 2 <= (int64_t)tile) tr++;
  while ((int64_t)tr * (tr + 1) / 2 > (int64_t)tile) tr--;
  const int tc = (int)(tile - (int64_t)tr * (tr + 1) / 2);
  const int q = d.q, n = d.d1, kq = gu_kq(q), K = single ? kq : 2 * kq, ks = 2 * kq + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const int i0 = tr * 64, l0 = tc * 64, wi = (wave >> 1) * 32, wl = (wave & 1) * 32;
  float* As = un_lds; float* Bs = un_lds + 64 * ks;
  auto outside = [&](int l) { return !(l >= g0 && l < g0 + q) && !(l >= j0 && l < j0 + q); };
  float old[2][2][4];
  auto at = [&](int a, int b, int r) { return (int64_t)(i0 + wi + a * 16 + 4 * lr + r) * n + l0 + wl + b * 16 + lc; };
  auto inside = [&](int a, int b, int r) {
    const int i = i0 + wi + a * 16 + 4 * lr + r, l = l0 + wl + b * 16 + lc;
    return i < n && l <= i;
  };
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 4; r++) old[a][b][r] = N[(int64_t)min(i0 + wi + a * 16 + 4 * lr + r, n - 1) * n + min(l0 + wl + b * 16 + lc, n - 1)];
  for (int half = 0; half < (single ? 1 : 2); half++) {
    stage_panel<64>(As, ks, half * kq, kq, (half ? P2D : P1D) + (int64_t)i0 * q, q, n - i0);
    stage_panel<64>(Bs, ks, half * kq, kq, (half ? P2 : P1) + (int64_t)l0 * q, q, n - l0);
  }
  __syncthreads();
  f4v acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++) acc[a][b] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int kk = 0; kk < K; kk += 4) {
    float av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; a++) { av[a] = As[(wi + a * 16 + lc) * ks + kk + lr]; bv[a] = Bs[(wl + a * 16 + lc) * ks + kk + lr]; }
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int b = 0; b < 2; b++) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (inside(a, b, r) && outside(i0 + wi + a * 16 + 4 * lr + r) && outside(l0 + wl + b * 16 + lc)) N[at(a, b, r)] = old[a][b][r] - acc[a][b][r];
}

// The state after the move: the pivots' rows of N (fix_blocks workgroups), Z and the columns' shares of the groups' Grams
// (p x chunks) and the bulk of N (its lower tiles), none of which reads what another writes, each after the acceptance test for
// itself; the first workgroup leaves the outcome in ctrl for the scores' launch.  As three launches after the one of the test:
// 4.5 + 10.2 + 6.3 us at 256 groups of 9 rows, 12.7 us as one, and a move is four launches, 40 us, instead of ten, 62 us.
// Bound by a pass over N and one over Z.
template <int RT>
__global__ __launch_bounds__(256, 2) void pair_state_kernel(TabDims d, float* __restrict__ N, float* __restrict__ Z, const float* __restrict__ P1,
                                                            const float* __restrict__ P2, const float* __restrict__ P1D,
                                                            const float* __restrict__ P2D, const float* __restrict__ rZ1,
                                                            const float* __restrict__ rZ2, const double* __restrict__ small, SearchCtrl* ctrl,
                                                            double* __restrict__ dblk, int32_t* __restrict__ kept, double* __restrict__ part,
                                                            const int32_t* __restrict__ single, int always_accept, const double* __restrict__ dpart,
                                                            int nparts, int fix_blocks, int chunk_cols, int chunks) {
  extern __shared__ float ps_lds[];
  if (ctrl->done) return;
  const int g = single ? *single : ctrl->g_out, j = single ? g : ctrl->g_in;
  double delta;
  const bool ok = pair_taken(ctrl, always_accept, dpart, nparts, delta);
  if (blockIdx.x == 0 && threadIdx.x == 0) { ctrl->delta = delta; ctrl->taken = ok; }
  if (!ok) return;
  const int b = blockIdx.x, groups = d.p * chunks;
  if (b < fix_blocks) pair_fix_rows<RT>(d, N, P1D, P2D, small, dblk, kept, single, g, j, b);
  else if (b < fix_blocks + groups)
    group_update<RT>(ps_lds, d, Z, P1, P2, rZ1, rZ2, small + 2 * d.q * d.q, single != nullptr, part, chunk_cols, chunks, g, j, (b - fix_blocks) / chunks,
                     (b - fix_blocks) % chunks);
  else update_N(ps_lds, d, N, P1, P2, P1D, P2D, single != nullptr, g * d.q, j * d.q, b - fix_blocks - groups);
}

// groups of one row: the float64 diagonal of the rows outside the pivots (theirs is written by pair_fix_rows)
__global__ __launch_bounds__(256) void pair_dblk_q1_kernel(TabDims d, const float* __restrict__ P1, const float* __restrict__ P2,
                                                            const float* __restrict__ P1D, const float* __restrict__ P2D,
                                                            const SearchCtrl* __restrict__ ctrl, double* __restrict__ dblk,
                                                            const int32_t* __restrict__ single) {
  if (ctrl->done) return;
  const int h = blockIdx.x * 256 + threadIdx.x, g = single ? *single : ctrl->g_out, j = single ? g : ctrl->g_in;
  if (h < d.p && h != g && h != j) dblk[h] -= (double)P1D[h] * (double)P1[h] + (double)P2D[h] * (double)P2[h];
}

// q = 1 fast path of the bulk update: N[i][l] -= a1[i]*b1[l] + a2[i]*b2[l] on the lower triangle.
// One workgroup streams a 32-row x 1024-column slab: each thread owns 4 consecutive columns and keeps their
// coefficients in registers while it walks down the rows.
__global__ __launch_bounds__(256) void update_N_q1_kernel(int n, float* __restrict__ N, const float* __restrict__ P1,
                                                           const float* __restrict__ P2, const float* __restrict__ P1D,
                                                           const float* __restrict__ P2D, const SearchCtrl* __restrict__ ctrl) {
  if (ctrl->done) return;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 1024;
  if (c0 > r0 + 31) return;
  const int c = c0 + threadIdx.x * 4;
  if (c >= n) return;
  const int rend = (r0 + 32 < n) ? r0 + 32 : n;
  if (c + 3 < n && (n & 3) == 0) {
    const float4 b1 = *reinterpret_cast<const float4*>(P1 + c);
    const float4 b2 = *reinterpret_cast<const float4*>(P2 + c);
#pragma unroll 4
    for (int i = r0; i < rend; i++) {
      if (c > i) continue;
      const float a1 = P1D[i], a2 = P2D[i];
      float4* p = reinterpret_cast<float4*>(N + (int64_t)i * n + c);
      float4 v = *p;
      v.x -= a1 * b1.x + a2 * b2.x;
      v.y -= a1 * b1.y + a2 * b2.y;
      v.z -= a1 * b1.z + a2 * b2.z;
      v.w -= a1 * b1.w + a2 * b2.w;
      *p = v;
    }
  } else {
    for (int i = r0; i < rend; i++)
      for (int u = 0; u < 4; u++) {
        int l = c + u;
        if (l < n && l <= i) N[(int64_t)i * n + l] -= P1D[i] * P1[l] + P2D[i] * P2[l];
      }
  }
}

// groups of one row: Z[i][:] -= P1[i] rZ1[:] + P2[i] rZ2[:], then gram[i] = |Z_i|^2
__global__ __launch_bounds__(256) void update_Z_kernel(TabDims d, float* __restrict__ Z, const float* __restrict__ P1,
                                                        const float* __restrict__ P2, const float* __restrict__ rZ1,
                                                        const float* __restrict__ rZ2, double* __restrict__ gram,
                                                        const SearchCtrl* __restrict__ ctrl) {
  if (ctrl->done) return;
  const int h = blockIdx.x, m = d.m;
  float* Zh = Z + (int64_t)h * m;
  {
    const float a1 = P1[h], a2 = P2[h];
    double v = 0;
    if ((m & 3) == 0) {                        // rows are 16-byte aligned: four columns per load
      float4* Z4 = reinterpret_cast<float4*>(Zh);
      const float4* r1 = reinterpret_cast<const float4*>(rZ1);
      const float4* r2 = reinterpret_cast<const float4*>(rZ2);
      for (int c4 = threadIdx.x; c4 < (m >> 2); c4 += 256) {
        float4 z = Z4[c4];
        const float4 x = r1[c4], y = r2[c4];
        z.x -= a1 * x.x + a2 * y.x; z.y -= a1 * x.y + a2 * y.y; z.z -= a1 * x.z + a2 * y.z; z.w -= a1 * x.w + a2 * y.w;
        Z4[c4] = z;
        v += (double)z.x * (double)z.x + (double)z.y * (double)z.y + (double)z.z * (double)z.z + (double)z.w * (double)z.w;
      }
    } else {
      for (int col = threadIdx.x; col < m; col += 256) {
        float z = Zh[col] - (a1 * rZ1[col] + a2 * rZ2[col]);
        Zh[col] = z;
        v += (double)z * (double)z;
      }
    }
    __shared__ double red[4];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) gram[h] = red[0] + red[1] + red[2] + red[3];
  }
}

// The `take` kept groups with the smallest removal cost (ascending cost, lowest index on ties) -> pick[0..take), and
// the relative gap between the costliest of them and the cheapest kept group left out -> *gap (inf if none is left).
// One workgroup; take <= 64.
// side 1: the same for the groups outside the kept set with the LARGEST addition gain (descending gain).
__global__ __launch_bounds__(1024) void greedy_pick_kernel(TabDims d, const int32_t* __restrict__ kept,
                                                            const double* __restrict__ score, int take,
                                                            int32_t* __restrict__ pick, float* __restrict__ gap,
                                                            const SearchCtrl* __restrict__ ctrl, int side) {
  __shared__ double s_v[1024];
  __shared__ int s_i[1024];
  __shared__ int chosen[65];
  __shared__ double chosen_v[65];
  if (side == 2) { side = blockIdx.x; pick += 64 * side; gap += side; }
  if (ctrl->done || ctrl->pause) return;
  const int tid = threadIdx.x;
  for (int round = 0; round <= take; round++) {
    double best = INFINITY;
    int ib = -1;
    for (int h = tid; h < d.p; h += 1024) {
      if ((kept[h] != 0) != (side == 0)) continue;
      bool used = false;
      for (int c = 0; c < round; c++) used |= (chosen[c] == h);
      if (used) continue;
      const double v = side ? -score[h] : score[h];
      if (ib < 0 || v < best) { best = v; ib = h; }        // ascending h per thread: strict comparison keeps the lowest index
    }
    s_v[tid] = best; s_i[tid] = ib;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
      if (tid < o) {
        const double b1 = s_v[tid + o]; const int ib2 = s_i[tid + o];
        const double a1 = s_v[tid]; const int ia = s_i[tid];
        if (ib2 >= 0 && (ia < 0 || b1 < a1 || (b1 == a1 && ib2 < ia))) { s_v[tid] = b1; s_i[tid] = ib2; }
      }
      __syncthreads();
    }
    if (tid == 0) { chosen[round] = s_i[0]; chosen_v[round] = s_v[0]; }
    __syncthreads();
  }
  if (tid < take) pick[tid] = chosen[tid];
  if (tid == 0) {
    const double edge = chosen_v[take - 1];
    *gap = (chosen[take] >= 0) ? (float)(fabs(chosen_v[take] - edge) / fmax(fabs(edge), 1e-300)) : INFINITY;
  }
}

// The same selection for p <= 1024 * KMAX groups with the eligible scores held in registers: every round is a local scan, a
// shuffle reduction per wave and one more over the 16 wave records, instead of another pass over memory.
// (value, index) of the smallest value, lowest index on ties (index -1: none), over the lanes of a row of 16, in all of them
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void best_step(double& v, int& i) {
  const int oi = __builtin_amdgcn_update_dpp(-1, i, CTRL, ROW_MASK, 0xF, false);
  const double ov = __hiloint2double(__builtin_amdgcn_update_dpp(0x7FF00000, __double2hiint(v), CTRL, ROW_MASK, 0xF, false),
                                     __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false));
  if (oi >= 0 && (i < 0 || ov < v || (ov == v && oi < i))) { v = ov; i = oi; }
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_or_inf(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0x7FF00000, __double2hiint(v), CTRL, ROW_MASK, 0xF, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ void best_of_16(double& v, int& i) {
  best_step<0xb1, 0xf>(v, i);      // quads: xor 1, xor 2
  best_step<0x4e, 0xf>(v, i);
  best_step<0x124, 0xf>(v, i);     // rows: rotate by 4, by 8
  best_step<0x128, 0xf>(v, i);
}
// ... over the wave, in lane 63
__device__ __forceinline__ void best_of_wave(double& v, int& i) {
  best_of_16(v, i);
  best_step<0x142, 0xa>(v, i);     // row 0 -> 1, 2 -> 3
  best_step<0x143, 0xc>(v, i);     // rows 0, 1 -> 2, 3
}
__device__ __forceinline__ double wave_least(double v) {      // in lane 63
  v = fmin(v, dpp_or_inf<0xb1, 0xf>(v)); v = fmin(v, dpp_or_inf<0x4e, 0xf>(v)); v = fmin(v, dpp_or_inf<0x124, 0xf>(v));
  v = fmin(v, dpp_or_inf<0x128, 0xf>(v)); v = fmin(v, dpp_or_inf<0x142, 0xa>(v)); v = fmin(v, dpp_or_inf<0x143, 0xc>(v));
  return v;
}
// The same from registers (p <= 1024 KMAX), one workgroup.  The least values of the 16 KMAX groups of 64 candidates are ranked by
// counting; the (take + 1)-th of them bounds the (take + 1)-th candidate, so the few candidates up to it are listed and ranked
// by counting as well: a fixed number of barriers whatever `take`.  Lists beyond PICK_CAP (many equal values, fewer groups than
// picks) are picked one by one: a thread keeps the best of its own candidates, a wave the best of its threads, a round merges the
// 16 waves' records in every wave and only the wave that lost its best looks for the next one.
constexpr int PICK_CAP = 128;
template <int KMAX>
__global__ __launch_bounds__(1024) void greedy_pick_reg_kernel(TabDims d, const int32_t* __restrict__ kept,
                                                                const double* __restrict__ score, int take,
                                                                int32_t* __restrict__ pick, float* __restrict__ gap,
                                                                const SearchCtrl* __restrict__ ctrl, int side) {
  constexpr int NG = 16 * KMAX, PARTS = 1024 / NG;
  __shared__ double w_v[2][16], g_v[NG], l_v[PICK_CAP], s_bound, s_edge[2];
  __shared__ int w_i[2][16], g_rank[NG], l_i[PICK_CAP], l_rank[PICK_CAP], s_n;
  if (side == 2) { side = blockIdx.x; pick += 64 * side; gap += side; }
  if (ctrl->done || ctrl->pause) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double v[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; k++) {
    const int h = tid + 1024 * k;
    v[k] = INFINITY;
    if (h < d.p && ((kept[h] != 0) == (side == 0))) v[k] = side ? -score[h] : score[h];
  }
#pragma unroll
  for (int k = 0; k < KMAX; k++) {
    const double least = wave_least(v[k]);
    if (lane == 63) g_v[k * 16 + wave] = least;
  }
  if (tid < NG) g_rank[tid] = 0;
  if (tid < PICK_CAP) l_rank[tid] = 0;
  if (tid == 0) { s_n = 0; s_bound = INFINITY; s_edge[0] = s_edge[1] = INFINITY; }
  __syncthreads();
  {
    const int e = tid % NG, j0 = tid / NG * (NG / PARTS);
    const double x = g_v[e];
    int below = 0;
#pragma unroll 8
    for (int j = j0; j < j0 + NG / PARTS; j++) below += g_v[j] < x || (g_v[j] == x && j < e);
    if (below) atomicAdd(&g_rank[e], below);
  }
  __syncthreads();
  if (tid < NG && g_rank[tid] == take) s_bound = g_v[tid];
  __syncthreads();
  const double bound = s_bound;
#pragma unroll
  for (int k = 0; k < KMAX; k++)
    if (v[k] <= bound && v[k] < INFINITY) {
      const int at = atomicAdd(&s_n, 1);
      if (at < PICK_CAP) { l_v[at] = v[k]; l_i[at] = tid + 1024 * k; }
    }
  __syncthreads();
  const int n = s_n;
  if (n <= PICK_CAP) {
    const int e = tid % PICK_CAP, j0 = tid / PICK_CAP * (PICK_CAP * PICK_CAP / 1024);
    if (e < n) {
      const double x = l_v[e];
      const int xi = l_i[e];
      int below = 0;
      for (int j = j0; j < min(n, j0 + PICK_CAP * PICK_CAP / 1024); j++) below += l_v[j] < x || (l_v[j] == x && l_i[j] < xi);
      if (below) atomicAdd(&l_rank[e], below);
    }
    __syncthreads();
    if (tid < n) {
      const int r = l_rank[tid];
      if (r < take) pick[r] = l_i[tid];
      if (r == take - 1) s_edge[0] = l_v[tid];
      if (r == take) s_edge[1] = l_v[tid];
    }
    if (tid >= n && tid < take) pick[tid] = -1;
    __syncthreads();
    if (tid == 0) *gap = n > take ? (float)(fabs(s_edge[1] - s_edge[0]) / fmax(fabs(s_edge[0]), 1e-300)) : INFINITY;
    return;
  }
  double best = INFINITY, prev = 0.0, edge = 0.0;
  int ib = -1, c = -1;
  for (int round = 0; round <= take; round++) {
    if (round == 0 || (c >= 0 && ((c & 1023) >> 6) == wave)) {      // uniform over the wave
      if (round == 0 || (c & 1023) == tid) {
        best = INFINITY; ib = -1;
#pragma unroll
        for (int k = 0; k < KMAX; k++) {
          if (round && k == (c >> 10)) v[k] = INFINITY;
          if (v[k] < best) { best = v[k]; ib = tid + 1024 * k; }      // ascending index per thread: strict comparison keeps the lowest
        }
      }
      double wb = best;
      int wi = ib;
      best_of_wave(wb, wi);
      if (lane == 63) { w_v[round & 1][wave] = wb; w_i[round & 1][wave] = wi; }
    } else if (lane == 63) {
      w_v[round & 1][wave] = w_v[(round & 1) ^ 1][wave]; w_i[round & 1][wave] = w_i[(round & 1) ^ 1][wave];
    }
    __syncthreads();
    double rb = w_v[round & 1][lane & 15];
    c = w_i[round & 1][lane & 15];
    best_of_16(rb, c);                                              // the same in every row of lanes of every wave
    prev = edge; edge = rb;
    if (tid == 0 && round < take) pick[round] = c;
  }
  if (tid == 0) *gap = (c >= 0) ? (float)(fabs(edge - prev) / fmax(fabs(prev), 1e-300)) : INFINITY;
}

hipError_t launch_greedy_pick(const TabDims& d, const TabPtrs& t, int take, int32_t* pick, float* gap, hipStream_t s, int side) {
  if (take < 1 || take > 64) return hipErrorInvalidValue;
  const dim3 grid(side == 2 ? 2 : 1);
  if (d.p <= 1024 * 8)
    hipLaunchKernelGGL(greedy_pick_reg_kernel<8>, grid, dim3(1024), 0, s, d, t.kept, t.score, take, pick, gap, t.ctrl, side);
  else if (d.p <= 1024 * 32)
    hipLaunchKernelGGL(greedy_pick_reg_kernel<32>, grid, dim3(1024), 0, s, d, t.kept, t.score, take, pick, gap, t.ctrl, side);
  else
    hipLaunchKernelGGL(greedy_pick_kernel, grid, dim3(1024), 0, s, d, t.kept, t.score, take, pick, gap, t.ctrl, side);
  return hipGetLastError();
}

hipError_t launch_select(const TabDims& d, const TabPtrs& t, int forced_out, int forced_in, hipStream_t s) {
  hipLaunchKernelGGL(select_kernel, dim3(1), dim3(1024), 0, s, d, t.kept, t.score, t.ctrl, forced_out, forced_in);
  return hipGetLastError();
}

hipError_t launch_search_iteration(const TabDims& d, const TabPtrs& t, int forced_out, int forced_in, int always_accept,
                                   hipStream_t s, hipEvent_t* ev, const int32_t* single, int exact_in) {
  const int q = d.q, rows64 = (d.d1 + 63) / 64;
  auto dynamic_lds = [](const void* kernel, size_t bytes, size_t beside) {
    return bytes + beside > 65536 ? hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) : hipSuccess;
  };
  int pick = single == nullptr;
  if (pick && d.p > PICK_MOST) {
    hipLaunchKernelGGL(select_kernel, dim3(1), dim3(1024), 0, s, d, t.kept, t.score, t.ctrl, forced_out, forced_in);
    pick = 0;
  }
  auto open = [&](int algebra) -> hipError_t {
    OSSCAR_BY_TILES(q, {
      const size_t lds = std::max((size_t)64 * 65 * 4, (size_t)q * (q + 1) * 28);
      const hipError_t e = dynamic_lds(reinterpret_cast<const void*>(pair_open_kernel<RT>), lds, sizeof(InvLds<RT>) + 1024);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(pair_open_kernel<RT>, dim3(4 * rows64 + algebra), dim3(256), lds, s, d, t.N, t.Z, t.kept, t.score, t.ctrl, t.C1, t.C2, t.rZ1, t.rZ2,
                         t.small, single, pick, forced_out, forced_in, algebra, rows64);
    })
    return hipGetLastError();
  };
  const int exact = exact_in && !single && forced_out < 0;
  hipError_t e = open(!exact);
  if (e != hipSuccess) return e;
  if (exact) {
    // the leaving group stands; choose the entering one by the exact gain of the pair and extract its panel again
    hipLaunchKernelGGL(exact_cross_kernel, dim3((d.d1 + 3) / 4), dim3(256), 0, s, d, t.Z, t.rZ1, t.ctrl, t.cross);
    if (q == 1) {
      hipLaunchKernelGGL(exact_q1_kernel, dim3((d.p + 255) / 256), dim3(256), 0, s, d, t.C1, t.cross, t.gram, t.dblk, t.kept, t.ctrl,
                         t.xscore);
    } else {
      const size_t xb_lds = (size_t)(3 * q * q + 256) * 8;
      e = dynamic_lds(reinterpret_cast<const void*>(exact_blocks_kernel), xb_lds, 0);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(exact_blocks_kernel, dim3(d.p), dim3(256), xb_lds, s, d, t.C1, t.cross, t.gram, t.dblk, t.kept, t.ctrl,
                         t.xgram, t.xdblk);
      launch_score(d, t.kept, t.xgram, t.xdblk, t.xscore, t.ctrl, 1, s);
    }
    hipLaunchKernelGGL(select_in_kernel, dim3(1), dim3(1024), 0, s, d, t.kept, t.xscore, t.ctrl);
    pick = 0;
    e = open(1);
    if (e != hipSuccess) return e;
  }
  // bulk panels go to C1D/C2D (times D) and to two further panels stored behind them
  float* P1 = t.C1D + (int64_t)2 * d.d1 * q;
  float* P2 = P1 + (int64_t)d.d1 * q;
  float* P1D = t.C1D;
  float* P2D = t.C2D;
  const int rows16 = (d.d1 + 15) / 16, ncb = (d.m + PC_COLS - 1) / PC_COLS;
  OSSCAR_BY_TILES(q, hipLaunchKernelGGL(pair_mid_kernel<RT>, dim3(rows16 + ncb), dim3(256), 0, s, d, t.C1, t.C2, t.small, t.ctrl, P1, P2, P1D, P2D,
                                        t.rZ1, t.rZ2, t.dpart, single, rows16))
  PairTrace tr;
  tr.out = t.trace_out; tr.in = t.trace_in; tr.gap = t.trace_gap; tr.obj = t.trace_obj;
  ScoreUpdate u;
  if (q == 1) {
    hipLaunchKernelGGL(pair_accept_kernel, dim3(1), dim3(64), 0, s, t.ctrl, always_accept, tr, single, t.dpart, ncb);
    hipLaunchKernelGGL(pair_fix_q1_kernel, dim3(rows16 + (d.m + 63) / 64), dim3(256), 0, s, d, t.N, t.Z, P1D, P2D, t.rZ1, t.rZ2, t.small, t.ctrl,
                       t.dblk, t.kept, single, rows16);
    if (ev) hipEventRecord(ev[0], s);
    hipLaunchKernelGGL(pair_dblk_q1_kernel, dim3((d.p + 255) / 256), dim3(256), 0, s, d, P1, P2, P1D, P2D, t.ctrl, t.dblk, single);
    dim3 grid((d.d1 + 1023) / 1024, (d.d1 + 31) / 32);
    hipLaunchKernelGGL(update_N_q1_kernel, grid, dim3(256), 0, s, d.d1, t.N, P1, P2, P1D, P2D, t.ctrl);
    if (ev) hipEventRecord(ev[1], s);
    hipLaunchKernelGGL(update_Z_kernel, dim3(d.p), dim3(256), 0, s, d, t.Z, P1, P2, t.rZ1, t.rZ2, t.gram, t.ctrl);
  } else {
    if (ev) hipEventRecord(ev[0], s);
    const int64_t tiles = (int64_t)rows64 * (rows64 + 1) / 2;
    const int cc = gu_chunk_cols(d.p, d.m), chunks = (d.m + cc - 1) / cc;
    OSSCAR_BY_TILES(q, {
      const size_t lds = std::max((size_t)2 * 64 * (2 * gu_kq(q) + 4) * 4, group_update_lds<RT>(gu_kq(q)));
      e = dynamic_lds(reinterpret_cast<const void*>(pair_state_kernel<RT>), lds, 2 * 16 * (16 * RT + 1) * 4);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(pair_state_kernel<RT>, dim3((unsigned)(rows16 + (int64_t)d.p * chunks + tiles)), dim3(256), lds, s, d, t.N, t.Z, P1, P2, P1D, P2D,
                         t.rZ1, t.rZ2, t.small, t.ctrl, t.dblk, t.kept, t.part, single, always_accept, t.dpart, ncb, rows16, cc, chunks);
    })
    if (ev) hipEventRecord(ev[1], s);
    u = ScoreUpdate{t.part, P1, P2, P1D, P2D, single, tr};
  }
  if (ev) hipEventRecord(ev[2], s);
  launch_score(d, t.kept, t.gram, t.dblk, t.score, t.ctrl, 1, s, u);
  return hipGetLastError();
}

}  // namespace osscar
