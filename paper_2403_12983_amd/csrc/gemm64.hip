// Float64-accumulating matrix products whose result is too small to fill the chip with 128 x 128 tiles, and the generic
// Gram products straight from the caller's rows.
//
//   C = alpha op(A) op(B) + beta Cin (+ diag_add on the diagonal), float64 sums on v_mfma_f64_16x16x4_f64
//
// 64 x 64 tiles (4 waves, 2 x 2 matrix-core tiles each) and, where there are few of them, the contraction cut into ranges
// that run as workgroups of ONE launch: each leaves its float64 tile in a workspace and a second kernel adds the ranges in
// index order, so the result does not depend on scheduling.  The matrix-core instruction takes 64 cycles for 2048 flops, so a
// wave's four products hide its four LDS reads and widening conversions, and the smaller tile costs nothing but L2 reads.
// What bounds these products is how many of the 256 compute units have work: the Gram of 288 columns is 15 tiles, which
// with one 128 x 128 tile per workgroup and the contraction in one piece took 0.65 ms for 4096 rows.
//
// An operand may be given with the contraction along its rows (K x rows, "k-major": the caller's activations X, whose Gram
// is X^T X), float32 or bf16, at any alignment.  A thread then takes one column and every fourth k, so that a wave reads 64
// neighbouring entries of one row; neither a transposed nor a float32 copy of X exists (they were a pass over memory of their
// own).  Patches of a feature map are written out as rows first (im2col_rows_kernel): gathered inside the product, once per
// tile that needs them, their addresses took longer than the matrix cores (2.8 ms against 1.5 for 12544 x 2304).
#include "internal.h"
#include <algorithm>
#include <type_traits>

namespace osscar {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int T64 = 64, KS = 32;
// LDS rows of 82 floats: the four k of a quarter-wave operand read start 18 banks apart, and the k-contiguous writes of a
// row-major operand (8 k apart between a row's four threads) 16 banks apart
constexpr int LD64 = 82;

struct Args64 {
  int M, N, K, kper, splits, tiles, tiles_n, lower, same;
  const void* A; int64_t lda; const void* B; int64_t ldb;
  double* part;                      // [split][tile][16][256] when splits > 1
  const void* Cin; int64_t ldcin; void* C; int64_t ldc;
  double alpha, beta, diag_add;
  int c_is_f64, vecA, vecB;
  const int *panels_m, *panels_n;
};

__device__ __forceinline__ void tile_of(const Args64& g, int t, int& tm, int& tn) {
  if (g.lower) {
    int r = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= t) r++;
    while (r * (r + 1) / 2 > t) r--;
    tm = r; tn = t - r * (r + 1) / 2;
  } else { tm = t / g.tiles_n; tn = t % g.tiles_n; }
}

__device__ __forceinline__ void emit(const Args64& g, int row, int col, double acc) {
  if (row >= g.M || col >= g.N) return;
  double v = g.alpha * acc;
  if (g.c_is_f64) {
    double* c = reinterpret_cast<double*>(g.C) + (int64_t)row * g.ldc + col;
    if (g.beta != 0.0) v += g.beta * reinterpret_cast<const double*>(g.Cin)[(int64_t)row * g.ldcin + col];
    if (row == col) v += g.diag_add;
    *c = v;
  } else {
    float* c = reinterpret_cast<float*>(g.C) + (int64_t)row * g.ldc + col;
    if (g.beta != 0.0) v += g.beta * (double)reinterpret_cast<const float*>(g.Cin)[(int64_t)row * g.ldcin + col];
    if (row == col) v += g.diag_add;
    *c = (float)v;
  }
}

// One operand's 64 x 32 stage, global memory -> registers (load: raw bits, addresses clamped into the operand) -> LDS (store:
// widened, zero outside).  Nothing of the loaded values is touched before store, so the loads stay in flight beside the products
// of the stage before.  KIND: see Opk64.
template <int KIND>
struct Loader {
  const float* pf; const uint16_t* ph; int64_t ld; int vec;
  int c, kq;                 // k-major: column of the tile, k = kq + 4 i
  int row, kk;               // row-major: row of the tile, k = kk .. kk + 8
  uint32_t raw[2][8];         // two stages in flight
  __device__ __forceinline__ Loader(const Args64& g, const void* p, int64_t ld_, int first, int rows, int vec_) {
    const int tid = threadIdx.x;
    ld = ld_; vec = vec_;
    c = tid & 63; kq = __builtin_amdgcn_readfirstlane(tid >> 6);
    row = tid >> 2; kk = (tid & 3) * 8;
    pf = reinterpret_cast<const float*>(p); ph = reinterpret_cast<const uint16_t*>(p);
    // rows (columns) past the end repeat the first one: they feed only elements that are never written
    if (KIND == OPK_ROW_F32) pf += (int64_t)(first + row < rows ? first + row : 0) * ld;
    else {
      const int col = first + c < rows ? first + c : 0;
      if (KIND == OPK_K_F32) pf += col;
      else ph += col;
    }
  }
  template <int U>
  __device__ __forceinline__ void load(const Args64& g, int k0, int kend) {
    if (KIND == OPK_ROW_F32) {
      const int k = k0 + kk;
      if (vec && k + 8 <= kend) {
        const uint4 a = *reinterpret_cast<const uint4*>(pf + k), b = *reinterpret_cast<const uint4*>(pf + k + 4);
        raw[U][0] = a.x; raw[U][1] = a.y; raw[U][2] = a.z; raw[U][3] = a.w; raw[U][4] = b.x; raw[U][5] = b.y; raw[U][6] = b.z; raw[U][7] = b.w;
      } else {
#pragma unroll
        for (int i = 0; i < 8; i++) raw[U][i] = __float_as_uint(pf[min(k + i, kend - 1)]);
      }
    } else if (KIND == OPK_K_F32 || KIND == OPK_K_BF16) {
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const int64_t o = (int64_t)min(k0 + kq + 4 * i, kend - 1) * ld;      // the same for the whole wave
        if (KIND == OPK_K_F32) raw[U][i] = __float_as_uint(pf[o]);
        else raw[U][i] = ph[o];
      }
    }
  }
  template <int U>
  __device__ __forceinline__ void store(float (*S)[LD64], int k0, int kend) const {
    const bool full = k0 + KS <= kend;      // uniform: only the last stage of a range has entries to clear
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const bool in = full || k0 + (KIND == OPK_ROW_F32 ? kk + i : kq + 4 * i) < kend;
      const uint32_t bits = KIND == OPK_K_BF16 ? raw[U][i] << 16 : raw[U][i];
      const float v = in ? __uint_as_float(bits) : 0.f;
      if (KIND == OPK_ROW_F32) S[kk + i][row] = v; else S[kq + 4 * i][c] = v;
    }
  }
};

template <int AK, int BK>
__global__ __launch_bounds__(256) void gemm64_kernel(Args64 g) {
  __shared__ float As[2][KS][LD64], Bs[2][KS][LD64];
  // ranges of the contraction go to the XCDs in turn (workgroup index modulo 8) when there are at least eight of them, so
  // that each XCD's L2 holds its own stretch of the operands
  int split, t;
  if (g.splits >= 8 && g.splits % 8 == 0) {
    const int b = blockIdx.x, grp = b / (8 * g.tiles), rest = b % (8 * g.tiles);
    split = grp * 8 + (rest & 7); t = rest >> 3;
  } else { split = blockIdx.x % g.splits; t = blockIdx.x / g.splits; }
  int tm, tn;
  tile_of(g, t, tm, tn);
  const int m0 = tm * T64, n0 = tn * T64;
  if (g.panels_m && !(g.panels_m[m0 >> 7] | g.panels_n[n0 >> 7])) return;
  const int kbeg = split * g.kper, kend = min(g.K, kbeg + g.kper);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  const bool one = g.same && tm == tn;            // a diagonal tile of A^T A: one operand serves as both
  Loader<AK> la(g, g.A, g.lda, m0, g.M, g.vecA);
  Loader<BK> lb(g, g.B, g.ldb, n0, g.N, g.vecB);
  d4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) acc[i][j] = d4{0, 0, 0, 0};
  auto load = [&](auto u, int k0) {
    la.template load<decltype(u)::value>(g, k0, kend);
    if (!one) lb.template load<decltype(u)::value>(g, k0, kend);
  };
  auto store = [&](auto u, int k0) {      // stage k0 into LDS buffer u
    la.template store<decltype(u)::value>(As[decltype(u)::value], k0, kend);
    if (!one) lb.template store<decltype(u)::value>(Bs[decltype(u)::value], k0, kend);
  };
  const std::integral_constant<int, 0> U0;
  const std::integral_constant<int, 1> U1;
  load(U0, kbeg);
  store(U0, kbeg);
  if (kbeg + KS < kend) load(U1, kbeg + KS);
  __syncthreads();
  // one stage: the loads of the stage after next are issued first, the next stage's (issued a stage ago) go to LDS at the end
  auto stage = [&](auto u, auto v, int k0) {
    constexpr int U = decltype(u)::value;
    if (k0 + 2 * KS < kend) load(u, k0 + 2 * KS);
    const float (*Ab)[LD64] = As[U];
    const float (*Bb)[LD64] = one ? As[U] : Bs[U];
#pragma unroll
    for (int s = 0; s < KS / 4; s++) {
      const int k = s * 4 + (lane >> 4);
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; i++) a[i] = (double)Ab[k][wm * 32 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 2; j++) b[j] = (double)Bb[k][wn * 32 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (k0 + KS < kend) store(v, k0 + KS);
    __syncthreads();
  };
  for (int k0 = kbeg; k0 < kend; k0 += 2 * KS) {
    stage(U0, U1, k0);
    if (k0 + KS < kend) stage(U1, U0, k0 + KS);
  }
  // lane holds D[4 r + lane/16][lane%16] of each 16 x 16 tile
  if (g.splits > 1) {
    double* p = g.part + ((int64_t)split * g.tiles + t) * 4096 + tid;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) p[((i * 2 + j) * 4 + r) * 256] = acc[i][j][r];
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) emit(g, m0 + wm * 32 + i * 16 + 4 * r + (lane >> 4), n0 + wn * 32 + j * 16 + (lane & 15), acc[i][j][r]);
}

// adds the ranges in index order: one thread per element, sixteen workgroups per tile, eight loads in flight
__global__ __launch_bounds__(256) void reduce64_kernel(Args64 g) {
  const int t = blockIdx.x >> 4, e = blockIdx.x & 15, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* p = g.part + (int64_t)t * 4096 + e * 256 + tid;
  const int64_t step = (int64_t)g.tiles * 4096;
  double v = 0;
  for (int s0 = 0; s0 < g.splits; s0 += 8) {
    double q[8];
#pragma unroll
    for (int u = 0; u < 8; u++) q[u] = (s0 + u < g.splits) ? p[(int64_t)(s0 + u) * step] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; u++) v += q[u];
  }
  int tm, tn;
  tile_of(g, t, tm, tn);
  const int i = e >> 3, j = (e >> 2) & 1, r = e & 3;
  emit(g, tm * T64 + (wave >> 1) * 32 + i * 16 + 4 * r + (lane >> 4), tn * T64 + (wave & 1) * 32 + j * 16 + (lane & 15), v);
}

template <int AK, int BK>
void start(const Args64& g, hipStream_t s) {
  hipLaunchKernelGGL((gemm64_kernel<AK, BK>), dim3((unsigned)(g.tiles * g.splits)), dim3(256), 0, s, g);
}

}  // namespace

static int gemm64_tiles(int M, int N, int lower) {
  const int tm = (M + T64 - 1) / T64, tn = (N + T64 - 1) / T64;
  return lower ? tm * (tm + 1) / 2 : tm * tn;
}

// Ranges of the contraction.  A stage of 32 k takes a workgroup that has its compute unit to itself about 1.7 us (the way of
// its loads) and every further one on the unit 0.9 - 1.05 us more (the matrix cores; two 2.65, three 3.6, four 4.7), so the time of a
// launch follows from the workgroups on the fullest unit and the stages of one; adding the ranges up costs a second launch and the
// write and read of their tiles (32 KB each).  Numbers of ranges timed one by one for 175 products (1 to 1128 tiles, K from 144 to 65536, all
// operand kinds): this rule is 0.8 % from the best on average.  With two and three workgroups on a unit at the same cost it was 3.5 %, and
// up to 23 % (1024 to 65536 rows of 440 to 640 columns, whose ranges then put three on a unit: 512 columns, 16384 rows 132 us in 16 ranges,
// 115 in 14); with no cost for the second one 3.1 %, up to 22 % (288 columns, 4096 rows 29.9 us in 22 ranges, 26.2 in 16).
static int gemm64_splits(int tiles, int K, size_t ws_bytes) {
  const int stages = std::max(1, (K + KS - 1) / KS);
  const int cap = (int)std::min<size_t>((size_t)stages, ws_bytes / ((size_t)tiles * 4096 * 8));
  int best = 1;
  double best_us = 1e30;
  for (int sp = 1; sp <= std::max(1, std::min(cap, 64)); sp++) {
    const int per = (stages + sp - 1) / sp, used = (stages + per - 1) / per;
    if (used != sp) continue;
    const int on_unit = (tiles * sp + 255) / 256;
    const double us = (1.75 + 0.9 * (on_unit - 1)) * per + (sp > 1 ? 3.0 + 0.018 * tiles * sp : 0.0);
    if (us < best_us * 0.98) { best_us = us; best = sp; }
  }
  return best;
}

hipError_t launch_gemm64(const Gemm64& q, hipStream_t s) {
  if (q.M <= 0 || q.N <= 0) return hipSuccess;
  Args64 g{};
  g.M = q.M; g.N = q.N; g.K = q.K; g.lower = q.lower; g.tiles_n = (q.N + T64 - 1) / T64; g.tiles = gemm64_tiles(q.M, q.N, q.lower);
  g.A = q.A; g.lda = q.lda; g.B = q.B; g.ldb = q.ldb;
  g.same = q.A == q.B && q.a_kind == q.b_kind && q.lda == q.ldb && q.a_kind != OPK_ROW_F32;
  g.Cin = q.Cin; g.ldcin = q.ldcin; g.C = q.C; g.ldc = q.ldc;
  g.alpha = q.alpha; g.beta = q.Cin ? q.beta : 0.0; g.diag_add = q.diag_add; g.c_is_f64 = q.c_is_f64;
  g.vecA = (q.lda % 4 == 0) && ((reinterpret_cast<uintptr_t>(q.A) & 15) == 0);
  g.vecB = (q.ldb % 4 == 0) && ((reinterpret_cast<uintptr_t>(q.B) & 15) == 0);
  const int stages = std::max(1, (q.K + KS - 1) / KS);
  g.panels_m = q.panels_m; g.panels_n = q.panels_n;
  g.splits = gemm64_splits(g.tiles, q.K, q.ws && !q.panels_m ? q.ws_bytes : 0);
  g.kper = (stages + g.splits - 1) / g.splits * KS;
  g.part = q.ws;
  switch (q.a_kind * 8 + q.b_kind) {
    case OPK_ROW_F32 * 8 + OPK_ROW_F32: start<OPK_ROW_F32, OPK_ROW_F32>(g, s); break;
    case OPK_ROW_F32 * 8 + OPK_K_F32: start<OPK_ROW_F32, OPK_K_F32>(g, s); break;
    case OPK_K_F32 * 8 + OPK_K_BF16: start<OPK_K_F32, OPK_K_BF16>(g, s); break;
    case OPK_K_F32 * 8 + OPK_K_F32: start<OPK_K_F32, OPK_K_F32>(g, s); break;
    case OPK_K_BF16 * 8 + OPK_K_BF16: start<OPK_K_BF16, OPK_K_BF16>(g, s); break;
    default: return hipErrorInvalidValue;
  }
  if (g.splits > 1) hipLaunchKernelGGL(reduce64_kernel, dim3((unsigned)g.tiles * 16), dim3(256), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gemm64_logged(const Gemm64& q, hipStream_t s) {
  int slot = -1;
  gemm_log_open(q.M, q.N, q.K, (q.c_is_f64 ? 2 : 0) | (q.lower ? 4 : 0) | (q.lower && q.A == q.B ? 8 : 0), s, &slot);
  const hipError_t e = launch_gemm64(q, s);
  gemm_log_close(slot, s);
  return e;
}

}  // namespace osscar
