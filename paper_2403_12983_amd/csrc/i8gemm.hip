// C = alpha A B + beta Cin for float32 operands, to the accuracy of float64 accumulation, on the int8 matrix cores.
//
// The large products of the state build (B = P G_K, V = P H_{K,Kc}, S, R of Proposition 4.1's closed forms and the
// residuals that refine them) need sums that are exact to far below float32 rounding; the float64 matrix-core
// instruction delivers that at 78.6 TFLOP/s, the int8 one runs 64 times as many multiply-adds per second.  Each row of A
// and each column of B is scaled by a power of two to (-1, 1) and cut into I8_S digits of 7 bits (signed, round to
// nearest: the first digit has 6 bits), x 2^-e = sum_t d_t 2^-(6 + 7 t), |d_t| <= 64, exactly while t < I8_S.  Products of
// digits are summed exactly in int32 (K 64^2 (t+1) < 2^31 for K < 100000), one accumulator set per digit weight
// g = t + u < I8_S: I8_S (I8_S + 1) / 2 = 15 integer products instead of one float64 product, and
//     C[i][j] = 2^(e_i + f_j) * sum_g acc_g[i][j] * 2^-(12 + 7 g)
// in float64.  What is dropped is below 2^-34 of (row maximum) x (column maximum) per term; on the 14336^3 products of the
// benchmark layer the result differs from the float64-accumulated one by 2e-9 of sum |a b|, the size of the float32
// rounding of the result itself.
// The digits are fixed-point relative to the largest entry of the row (column), so an entry 2^-b of that maximum keeps
// 34 - b bits.  The inverse P of a Gram matrix has a diagonal 10^3 - 10^4 times its off-diagonal entries, which would leave
// those with about 21 bits and, through the cancellation in P H_{K,Kc}, a 5e-5 error in V.  So a square operand can have its
// diagonal taken out (diag_a, diag_b): the diagonal is left out of the scaling and the digits, and its term A_ii B_ij
// (A_ij B_jj) is added in float64 in the epilogue.  Likewise along the contraction: the rows and columns of a Gram matrix
// scale with s_k = sqrt(H_kk), those of its inverse with 1 / s_k, so an outlier channel (s_k 20 times the rest) would cost the
// other entries of every row that crosses it 4 - 9 bits.  With kexp[k] = round(log2 s_k) the product is computed as
// (A 2^(+-kexp)) (2^(-+kexp) B), exact scalings that level both operands along k (ksign = +1: A inverse-like, B Gram-like).
//
// Layout of a packed operand: packet (16 consecutive k of one row, one digit) at
//     ((panel * nstages + stage) * I8_S + t) * 256 + kh * 128 + r,   panel = row / 128, stage = k / 32, kh = (k % 32) / 16, r = row % 128,
// so a (stage, panel) block of I8_S * 4 KB is the A- or B-side input of one v_mfma_i32_32x32x32_i8 step of a 128-row tile.
// The kernel: one workgroup of 8 waves (two per SIMD) per 128 x 128 tile, wave tile 64 x 32 = 2 matrix-core tiles x I8_S
// accumulator sets (160 registers); operand blocks go from global memory straight into LDS (global_load_lds_dwordx4), three
// stage buffers, loads three stages ahead; one barrier per stage that waits for LDS traffic only, placed before the last
// two products of the stage so that the next stage's row-side operands are on their way while those run.  14336^3: 36.2 ms
// (0.49 of the int8 peak); 42.0 ms while the compiler's own waits emptied the request queue every stage.  (4 waves of 64 x 64, one
// per SIMD, took 51 ms where 8 took 41: nothing to run while a wave waits.)
#include "internal.h"
#include <algorithm>

namespace osscar {
namespace {
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
constexpr int S = I8_S;

__device__ __forceinline__ int expo_of(unsigned bits) {      // smallest e with v < 2^e (0 for v = 0)
  const float v = __uint_as_float(bits);
  if (!(v > 0.f) || bits >= 0x7F800000u) return 0;
  int e;
  frexpf(v, &e);
  return max(e, -120);      // below, 2^-e would leave float32's range
}

// mx[r] = bit pattern of max |X[r, :]| (non-negative floats order like their bit patterns)
__global__ __launch_bounds__(256) void i8_absmax_rows_kernel(const float* __restrict__ X, int R, int K, int64_t ld, int skip_diag,
                                                              const int* __restrict__ kexp, int ks, unsigned* __restrict__ mx) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= R) return;
  float v = 0.f;
  for (int kb = 0; kb < K; kb += 512) {      // eight loads in flight; past the end the last column again, which changes no maximum
    float x[8];
    int e[8];
#pragma unroll
    for (int u = 0; u < 8; u++) { const int k = min(kb + 64 * u + lane, K - 1); x[u] = X[(int64_t)row * ld + k]; e[u] = kexp ? kexp[k] : 0; }
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const float a = fabsf(ldexpf(x[u], ks * e[u]));
      v = fmaxf(v, skip_diag && min(kb + 64 * u + lane, K - 1) == row ? 0.f : a);
    }
  }
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  if (lane == 0) mx[row] = __float_as_uint(v);
}
// mx[c] = max over the rows [64 y, 64 y + 64) of |X[:, c]|, joined by an atomic maximum (order-independent); mx zeroed before.  Sixteen loads
// in flight: one at a time, 256 rows of it, a matrix of 1152 columns took 71 us and one of 4096 115.
constexpr int AC_ROWS = 64;
__global__ __launch_bounds__(256) void i8_absmax_cols_kernel(const float* __restrict__ X, int K, int N, int64_t ld, int skip_diag,
                                                              const int* __restrict__ kexp, int ks, unsigned* __restrict__ mx) {
  const int col = blockIdx.x * 256 + threadIdx.x, cc = min(col, N - 1), k0 = blockIdx.y * AC_ROWS;
  float v = 0.f;
  for (int kb = k0; kb < min(K, k0 + AC_ROWS); kb += 16) {      // past the end the last row again, which changes no maximum
    float x[16];
    int e[16];
#pragma unroll
    for (int u = 0; u < 16; u++) { const int k = min(kb + u, K - 1); x[u] = X[(int64_t)k * ld + cc]; e[u] = kexp ? kexp[k] : 0; }
#pragma unroll
    for (int u = 0; u < 16; u++) {
      const float a = fabsf(ldexpf(x[u], ks * e[u]));
      v = fmaxf(v, skip_diag && min(kb + u, K - 1) == col ? 0.f : a);
    }
  }
  if (col < N) atomicMax(&mx[col], __float_as_uint(v));
}
__global__ void i8_zero_kernel(unsigned* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// 16 scaled values -> S packets of 16 digits each (every step is exact in float32)
template <int S>
__device__ __forceinline__ void slice16(const float* v, uint4* out) {
  unsigned w[S][4];
#pragma unroll
  for (int t = 0; t < S; t++) { w[t][0] = w[t][1] = w[t][2] = w[t][3] = 0u; }
#pragma unroll
  for (int j = 0; j < 16; j++) {
    float r = v[j] * 64.f;
#pragma unroll
    for (int t = 0; t < S; t++) {
      const float d = rintf(r);
      w[t][j >> 2] |= ((unsigned)((int)d & 0xff)) << (8 * (j & 3));
      r = (r - d) * 128.f;
    }
  }
#pragma unroll
  for (int t = 0; t < S; t++) out[t] = uint4{w[t][0], w[t][1], w[t][2], w[t][3]};
}

// A-side: X is R x K, the contraction runs along a row.  64 rows x 64 k per workgroup through LDS, so that reads run along the
// rows at any alignment and writes along the rows of a packet column (5461 x 5461 at odd alignment: 0.48 ms as 16 strided
// loads per thread).
__global__ __launch_bounds__(256) void i8_pack_rows_kernel(const float* __restrict__ X, int R, int K, int64_t ld, int skip_diag,
                                                            const int* __restrict__ kexp, int ks, const unsigned* __restrict__ mx, uint4* __restrict__ out,
                                                            int nstages) {
  __shared__ float T[64][65];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.y * 64, k = blockIdx.x * 64 + lane;
  const int e = (kexp && k < K) ? ks * kexp[k] : 0;
#pragma unroll 8
  for (int i = 0; i < 16; i++) {
    const int r = wave + 4 * i, row = row0 + r;
    float v = 0.f;
    if (row < R && k < K && !(skip_diag && k == row)) {
      v = X[(int64_t)row * ld + k] * ldexpf(1.f, -expo_of(mx[row]));
      if (kexp) v = ldexpf(v, e);
    }
    T[r][lane] = v;
  }
  __syncthreads();
  const int kp = blockIdx.x * 4 + wave, row = row0 + lane;      // a wave: one packet column of 64 rows
  if (kp >= nstages * 2) return;
  float v[16];
#pragma unroll
  for (int j = 0; j < 16; j++) v[j] = T[lane][wave * 16 + j];
  uint4 pk[S];
  slice16<S>(v, pk);
  const int stage = kp >> 1, kh = kp & 1, panel = row >> 7, r = row & 127;
#pragma unroll
  for (int t = 0; t < S; t++) out[(((int64_t)panel * nstages + stage) * S + t) * 256 + kh * 128 + r] = pk[t];
}
// B-side: X is K x N, the contraction runs down a column.  Thread = (packet of 16 k, column), columns fastest.
__global__ __launch_bounds__(256) void i8_pack_cols_kernel(const float* __restrict__ X, int K, int N, int64_t ld, int skip_diag,
                                                            const int* __restrict__ kexp, int ks, const unsigned* __restrict__ mx, uint4* __restrict__ out, int npanels,
                                                            int nstages) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int cpad = npanels * 128;
  const int kp = (int)(idx / cpad), col = (int)(idx % cpad);
  if (kp >= nstages * 2) return;
  float v[16];
#pragma unroll
  for (int j = 0; j < 16; j++) v[j] = 0.f;
  if (col < N) {
    const float sc = ldexpf(1.f, -expo_of(mx[col]));
#pragma unroll
    for (int j = 0; j < 16; j++)
      if (kp * 16 + j < K && !(skip_diag && kp * 16 + j == col))
        v[j] = ldexpf(X[(int64_t)(kp * 16 + j) * ld + col], kexp ? ks * kexp[kp * 16 + j] : 0) * sc;
  }
  uint4 pk[S];
  slice16<S>(v, pk);
  const int stage = kp >> 1, kh = kp & 1, panel = col >> 7, r = col & 127;
#pragma unroll
  for (int t = 0; t < S; t++) out[(((int64_t)panel * nstages + stage) * S + t) * 256 + kh * 128 + r] = pk[t];
}

}  // namespace
// kexp[k] = round(log2 sqrt(D[k][k])) for a positive diagonal, 0 otherwise (clamped to +-60)
__global__ void i8_kexp_kernel(const float* __restrict__ D, int n, int64_t ld, int* __restrict__ kexp) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const float d = D[(int64_t)k * ld + k];
  int e = 0;
  if (d > 0.f && d < 3e38f) e = (int)rintf(0.5f * log2f(d));
  kexp[k] = max(-60, min(60, e));
}
hipError_t launch_i8_kexp(const float* D, int n, int64_t ld, int* kexp, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(i8_kexp_kernel, dim3((n + 255) / 256), dim3(256), 0, s, D, n, ld, kexp);
  return hipGetLastError();
}
namespace {
struct I8Args {
  const uint4* Ap; const uint4* Bp; int nstages;
  const unsigned* mxa; const unsigned* mxb;
  const float* Cin; int64_t ldcin; float* C; int64_t ldc;
  int M, N, tiles_m, tiles_n, lower_only;
  double alpha, beta, diag_add;
  const float* A; int64_t lda; const float* B; int64_t ldb; int diag_a, diag_b;      // the operands themselves, for the diagonal terms
  double* C64;      // set: C64[row][col] += A B (leading dimension ldc, lower_only: on and below the diagonal) instead of C
  const int* skip_a; const int* skip_b;      // with C64: tiles of these row or column panels are left to another kernel
};

// vmcnt <= N; lgkmcnt = 0, then the barrier: builtins, which the compiler takes into account where it places waits of its own
template <int N>
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14)); }
__device__ __forceinline__ void lds_only_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int S>      // digits per operand (4 or 5)
__global__ __launch_bounds__(512, 1) void i8_gemm_kernel(I8Args g) {
  constexpr int BLK = S * 256;                   // packets of one (stage, panel) block
  constexpr int NG = 5;                          // digit weights t + u < NG that are summed, one accumulator set each
  constexpr int NL = NG - S + 1;                 // row-side digits that the last column-side digit meets
  // Stage buffers, each the A block followed by the B block.  Three arrays and a steady loop without conditions: with one
  // array, or with conditional requests, the compiler cannot tell which requests a read of LDS depends on and waits for all
  // of them, the one just issued for three stages later included.
  __shared__ uint4 lb0[2 * BLK], lb1[2 * BLK], lb2[2 * BLK];
  // 8 x 8 super-blocks of tiles, dealt to the XCDs in turn (workgroup index modulo 8): the tiles an XCD works on together
  // share row and column panels in its L2.  lower_only: the super-blocks on or below the diagonal.
  int tm, tn;
  {
    const int b = blockIdx.x, xcd = b & 7, slot = b >> 3;
    const int sbi = (slot / 64) * 8 + xcd, within = slot % 64;
    if (g.lower_only) {
      const int nr = (g.tiles_m + 7) / 8;
      if (sbi >= nr * (nr + 1) / 2) return;
      int r = (int)((sqrtf(8.f * (float)sbi + 1.f) - 1.f) * 0.5f);
      while ((r + 1) * (r + 2) / 2 <= sbi) r++;
      while (r * (r + 1) / 2 > sbi) r--;
      tm = r * 8 + within / 8;
      tn = (sbi - r * (r + 1) / 2) * 8 + within % 8;
      if (tm >= g.tiles_m || tn > tm) return;
    } else {
      const int nsb_c = (g.tiles_n + 7) / 8, nsb = ((g.tiles_m + 7) / 8) * nsb_c;
      if (sbi >= nsb) return;
      tm = (sbi / nsb_c) * 8 + within / 8;
      tn = (sbi % nsb_c) * 8 + within % 8;
      if (tm >= g.tiles_m || tn >= g.tiles_n) return;
    }
  }
  if (g.skip_a && (g.skip_a[tm] | g.skip_b[tn])) return;
  const int nstages = g.nstages;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 2, wn = wave & 3;      // wave tile: 64 rows x 32 columns
  v16i acc[NG][2];
#pragma unroll
  for (int q = 0; q < NG; q++)
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[q][a][r] = 0;
  const uint4* ga = g.Ap + (int64_t)tm * nstages * BLK;
  const uint4* gb = g.Bp + (int64_t)tn * nstages * BLK;
  // A stage is the A block followed by the B block, 2 BLK packets; instruction i of a wave moves packets
  // [512 i + 64 wave, + 64) (the boundary BLK is a multiple of 64: a wave's 64 lie in one block); lane l's 16 bytes
  // land at the LDS base + 16 l.
  constexpr int NI = (2 * BLK) / 512;
  static_assert(BLK % 256 == 0, "every wave issues the same number of loads per stage");
#define OSSCAR_I8_ISSUE(st_, buf_)                                                                                               \
  {                                                                                                                              \
    _Pragma("unroll") for (int i = 0; i < NI; i++) {                                                                             \
      const int p0 = i * 512 + wave * 64;                                                                                        \
      const uint4* src = (p0 < BLK) ? ga + (int64_t)(st_) * BLK + p0 + lane : gb + (int64_t)(st_) * BLK + (p0 - BLK) + lane;     \
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,                                       \
                                       (__attribute__((address_space(3))) void*)(buf_ + p0), 16, 0, 0);                          \
    }                                                                                                                            \
  }
#define OSSCAR_I8_READ_A(buf_)                                                                                                   \
  _Pragma("unroll") for (int t = 0; t < S; t++) _Pragma("unroll") for (int a = 0; a < 2; a++) {                                  \
    uint4 q = buf_[t * 256 + oa + a * 32];                                                                                       \
    fa[a][t] = *reinterpret_cast<v4i*>(&q);                                                                                      \
  }
  // A stage: column-side digits 0 .. S-2 against every row-side digit they meet (28 of its 30 products, 22 of 26 with four
  // digits).  The last
  // column-side digit goes to a register; then every wave has taken all it needs from this stage's buffer, which the barrier
  // establishes, and NEXT refills the buffer with the stage three ahead and requests the next stage's row-side operands
  // before the last two products.
#define OSSCAR_I8_STAGE(cur_, NEXT)                                                                                              \
  {                                                                                                                              \
    const uint4* pb = cur_ + BLK;                                                                                                \
    _Pragma("unroll") for (int u = 0; u < S - 1; u++) {                                                                          \
      v4i fb;                                                                                                                    \
      { uint4 q = pb[u * 256 + ob]; fb = *reinterpret_cast<v4i*>(&q); }                                                          \
      _Pragma("unroll") for (int t = 0; t < S && t + u < NG; t++) _Pragma("unroll") for (int a = 0; a < 2; a++)                  \
        acc[t + u][a] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a][t], fb, acc[t + u][a], 0, 0, 0);                             \
    }                                                                                                                            \
    v4i fl;                                                                                                                      \
    { uint4 q = pb[(S - 1) * 256 + ob]; fl = *reinterpret_cast<v4i*>(&q); }                                                      \
    v4i a0[2][NL];                                                                                                               \
    _Pragma("unroll") for (int t = 0; t < NL; t++) { a0[0][t] = fa[0][t]; a0[1][t] = fa[1][t]; }                                 \
    NEXT                                                                                                                         \
    _Pragma("unroll") for (int t = 0; t < NL; t++) _Pragma("unroll") for (int a = 0; a < 2; a++)                                 \
      acc[S - 1 + t][a] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0[a][t], fl, acc[S - 1 + t][a], 0, 0, 0);                       \
  }
#define OSSCAR_I8_STEADY(st_, cur_, nxt_)                                                                                        \
  OSSCAR_I8_STAGE(cur_, wait_loads<NI>(); lds_only_barrier(); OSSCAR_I8_ISSUE((st_) + 3, cur_); OSSCAR_I8_READ_A(nxt_))
#define OSSCAR_I8_TAIL(st_, cur_, nxt_)                                                                                          \
  if ((st_) < nstages)                                                                                                           \
    OSSCAR_I8_STAGE(cur_, if ((st_) + 1 < nstages) {                                                                             \
      wait_loads<0>(); lds_only_barrier();                                                                                       \
      if ((st_) + 3 < nstages) OSSCAR_I8_ISSUE((st_) + 3, cur_);                                                                 \
      OSSCAR_I8_READ_A(nxt_)                                                                                                     \
    })
  const int oa = (lane >> 5) * 128 + wm * 64 + (lane & 31), ob = (lane >> 5) * 128 + wn * 32 + (lane & 31);
  OSSCAR_I8_ISSUE(0, lb0);
  if (nstages > 1) OSSCAR_I8_ISSUE(1, lb1);
  if (nstages > 2) OSSCAR_I8_ISSUE(2, lb2);
  // stage 0 has landed (each wave waits for its own loads of that stage, then the barrier)
  if (nstages > 2) wait_loads<2 * NI>(); else wait_loads<0>();
  lds_only_barrier();
  v4i fa[2][S];
  OSSCAR_I8_READ_A(lb0)
  int st = 0;
  if (nstages >= 6) {
    do {
      OSSCAR_I8_STEADY(st, lb0, lb1)
      OSSCAR_I8_STEADY(st + 1, lb1, lb2)
      OSSCAR_I8_STEADY(st + 2, lb2, lb0)
      st += 3;
    } while (st + 6 <= nstages);
  }
  for (; st < nstages; st += 3) {
    OSSCAR_I8_TAIL(st, lb0, lb1)
    OSSCAR_I8_TAIL(st + 1, lb1, lb2)
    OSSCAR_I8_TAIL(st + 2, lb2, lb0)
  }
#undef OSSCAR_I8_ISSUE
#undef OSSCAR_I8_READ_A
#undef OSSCAR_I8_STAGE
#undef OSSCAR_I8_STEADY
#undef OSSCAR_I8_TAIL
  // C layout of a 32 x 32 tile: register r = rr*4 + r3 holds row rr*8 + (lane/32)*4 + r3, column lane%32
  const int col = tn * 128 + wn * 32 + (lane & 31);
  const int eb = expo_of(g.mxb[col < g.N ? col : 0]);
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int row = tm * 128 + wm * 64 + a * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      if (row < g.M && col < g.N) {
        if (g.C64) {      // the same digits, plain sum
          double v = 0.0;
#pragma unroll
          for (int q = NG - 1; q >= 0; q--) v = v * (1.0 / 128.0) + (double)acc[q][a][r];
          v = ldexp(v, expo_of(g.mxa[row]) + eb - 12);
          if (!g.lower_only || col <= row) g.C64[(int64_t)row * g.ldc + col] += v;
          continue;
        }
        double v = 0.0;
#pragma unroll
        for (int q = NG - 1; q >= 0; q--) v = v * (1.0 / 128.0) + (double)acc[q][a][r];
        v = ldexp(v, expo_of(g.mxa[row]) + eb - 12);
        // the diagonal terms that were left out of the digits: k = row of A (A square), k = col of B (B square)
        if (g.diag_a) v += (double)g.A[(int64_t)row * g.lda + row] * (double)g.B[(int64_t)row * g.ldb + col];
        if (g.diag_b && !(g.diag_a && row == col)) v += (double)g.A[(int64_t)row * g.lda + col] * (double)g.B[(int64_t)col * g.ldb + col];
        v *= g.alpha;
        if (g.beta != 0.0) v += g.beta * (double)g.Cin[(int64_t)row * g.ldcin + col];
        if (row == col) v += g.diag_add;
        g.C[(int64_t)row * g.ldc + col] = (float)v;
      }
    }
}
}  // namespace

size_t i8_pack_bytes(int64_t rows, int64_t K) {
  return (size_t)S * 16 * (size_t)((rows + 127) / 128 * 128) * (size_t)((K + 31) / 32 * 2);
}

bool i8_gemm_fits(const GemmArgs& g) {
  // int32 sums: K * 64^2 * S must stay below 2^31; float32 in and out, plain A B
  return g.M > 0 && g.N > 0 && g.K > 0 && g.K <= 100000 && !g.c_is_f64 && !g.trans_b && !g.acc_f32 && (g.beta == 0.0 || g.Cin != nullptr);
}

hipError_t launch_i8_gemm(const GemmArgs& g, void* packA, size_t capA, void* packB, size_t capB, unsigned* mx, size_t mx_entries,
                          hipStream_t s) {
  if (!i8_gemm_fits(g) || (g.lower_only && g.M != g.N)) return hipErrorInvalidValue;
  if ((g.i8_diag_a && g.M != g.K) || (g.i8_diag_b && g.N != g.K)) return hipErrorInvalidValue;
  if (g.i8_kexp && g.i8_ksign != 1 && g.i8_ksign != -1) return hipErrorInvalidValue;
  if (i8_pack_bytes(g.M, g.K) > capA || i8_pack_bytes(g.N, g.K) > capB || (size_t)g.M + (size_t)g.N > mx_entries) return hipErrorInvalidValue;
  if ((reinterpret_cast<uintptr_t>(packA) & 15) || (reinterpret_cast<uintptr_t>(packB) & 15)) return hipErrorInvalidValue;
  const int npa = (g.M + 127) / 128, npb = (g.N + 127) / 128, nst = (g.K + 31) / 32;
  unsigned* mxa = mx; unsigned* mxb = mx + g.M;
  int log_slot = -1;
  gemm_log_open(g.M, g.N, g.K, 16 | (g.lower_only ? 4 : 0), s, &log_slot);
  hipLaunchKernelGGL(i8_zero_kernel, dim3((g.N + 255) / 256), dim3(256), 0, s, mxb, g.N);
  hipLaunchKernelGGL(i8_absmax_rows_kernel, dim3((g.M + 3) / 4), dim3(256), 0, s, g.A, g.M, g.K, g.lda, g.i8_diag_a, g.i8_kexp, g.i8_ksign, mxa);
  hipLaunchKernelGGL(i8_absmax_cols_kernel, dim3((g.N + 255) / 256, (g.K + AC_ROWS - 1) / AC_ROWS), dim3(256), 0, s, g.B, g.K, g.N, g.ldb, g.i8_diag_b, g.i8_kexp, -g.i8_ksign, mxb);
  hipLaunchKernelGGL(i8_pack_rows_kernel, dim3((unsigned)((nst + 1) / 2), (unsigned)(npa * 2)), dim3(256), 0, s, g.A, g.M, g.K, g.lda, g.i8_diag_a, g.i8_kexp,
                     g.i8_ksign, mxa, reinterpret_cast<uint4*>(packA), nst);
  hipLaunchKernelGGL(i8_pack_cols_kernel, dim3((unsigned)(((int64_t)nst * 2 * npb * 128 + 255) / 256)), dim3(256), 0, s, g.B, g.K, g.N, g.ldb,
                     g.i8_diag_b, g.i8_kexp, -g.i8_ksign, mxb, reinterpret_cast<uint4*>(packB), npb, nst);
  I8Args a{};
  a.Ap = reinterpret_cast<const uint4*>(packA); a.Bp = reinterpret_cast<const uint4*>(packB); a.nstages = nst;
  a.mxa = mxa; a.mxb = mxb; a.Cin = g.Cin; a.ldcin = g.ldcin; a.C = reinterpret_cast<float*>(g.C); a.ldc = g.ldc;
  a.M = g.M; a.N = g.N; a.tiles_m = npa; a.tiles_n = npb; a.lower_only = g.lower_only;
  a.alpha = g.alpha; a.beta = g.beta; a.diag_add = g.diag_add;
  a.A = g.A; a.lda = g.lda; a.B = g.B; a.ldb = g.ldb; a.diag_a = g.i8_diag_a; a.diag_b = g.i8_diag_b;
  int nsb;
  if (g.lower_only) { const int nr = (npa + 7) / 8; nsb = nr * (nr + 1) / 2; }
  else nsb = ((npa + 7) / 8) * ((npb + 7) / 8);
  hipLaunchKernelGGL(i8_gemm_kernel<S>, dim3((unsigned)((nsb + 7) / 8 * 8 * 64)), dim3(512), 0, s, a);
  gemm_log_close(log_slot, s);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// C64 (M x N float64) += X^T Y (Y == nullptr: X^T X, lower triangle) for rows of float32 or bf16 at any alignment: both operands
// are packed as B-side operands, digits relative to their column's largest value in this call: float32 five digits, so a value is
// carried to 2^-35 of the maximum; bf16 four (13 products), so a value within 2^-18 of the maximum is carried whole.  Products
// of digits t + u >= 5 are dropped: unequal digits first, whose signs are independent; dropped squares start at t + u = 6, at most
// 2^-42 of the maximum's square per row, 2^-28 over 16384 rows.  (With four digits and t + u < 4 alone a diagonal came out 5e-6
// off.)  All that is relative to the two columns' maxima, while H is of the size of their norms: for 7777 rows
// of independent normal values the 2-norm of H's error off the diagonal is 2.529e-8 of H, 2.528e-8 with float64 sums (both
// float32's rounding of H), but 1.3e-7 with one value of 100 sigma in every column.  So a column counts, while it is packed, its
// nonzero values and the squares of their first digits; if their rms is below 1/16 of the power of two above the maximum (normal
// values: 1/8 or more; the dropped products grow with the square), or if a value is not finite, its panel of 128 columns is
// left out here and the caller forms the tiles that it takes part in with float64 sums.
// ------------------------------------------------------------------------------------------------
namespace {
__device__ __forceinline__ float load_as_float(const float* p) { return *p; }
__device__ __forceinline__ float load_as_float(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }
// mx[c] = largest bit pattern of |X[:, c]| over the rows [128 y, 128 y + 128): infinities and NaN stand above every number
template <typename T>
__global__ __launch_bounds__(256) void i8_absbits_cols_kernel(const T* __restrict__ X, int K, int N, int64_t ld, unsigned* __restrict__ mx) {
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= N) return;
  const int k0 = blockIdx.y * 128, k1 = min(K, k0 + 128);
  unsigned v = 0u;
#pragma unroll 8
  for (int k = k0; k < k1; k++) v = max(v, __float_as_uint(load_as_float(X + (int64_t)k * ld + col)) & 0x7FFFFFFFu);
  atomicMax(&mx[col], v);
}
template <int S, typename T>
__global__ __launch_bounds__(256) void i8_pack_rows_of_x_kernel(const T* __restrict__ X, int K, int N, int64_t ld, const unsigned* __restrict__ mx,
                                                                 unsigned long long* __restrict__ stat, uint4* __restrict__ out, int npanels, int nstages) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int cpad = npanels * 128;
  const int kp = (int)(idx / cpad), col = (int)(idx % cpad);
  if (kp >= nstages * 2) return;
  float v[16];
#pragma unroll
  for (int j = 0; j < 16; j++) v[j] = 0.f;
  if (col < N && mx[col] < 0x7F800000u) {
    const int e = expo_of(mx[col]);
#pragma unroll
    for (int j = 0; j < 16; j++)
      if (kp * 16 + j < K) v[j] = ldexpf(load_as_float(X + (int64_t)(kp * 16 + j) * ld + col), -e);
  }
  uint4 pk[S];
  slice16<S>(v, pk);
  int nonzero = 0, squares = 0;      // squares of the first digits: 16384 rows of 64^2 fit
#pragma unroll
  for (int j = 0; j < 16; j++) nonzero += v[j] != 0.f;
  squares = __builtin_amdgcn_sdot4((int)pk[0].x, (int)pk[0].x, squares, false);
  squares = __builtin_amdgcn_sdot4((int)pk[0].y, (int)pk[0].y, squares, false);
  squares = __builtin_amdgcn_sdot4((int)pk[0].z, (int)pk[0].z, squares, false);
  squares = __builtin_amdgcn_sdot4((int)pk[0].w, (int)pk[0].w, squares, false);
  if (nonzero) atomicAdd(&stat[col], ((unsigned long long)nonzero << 32) + (unsigned)squares);
  const int stage = kp >> 1, kh = kp & 1, panel = col >> 7, r = col & 127;
#pragma unroll
  for (int t = 0; t < S; t++) out[(((int64_t)panel * nstages + stage) * S + t) * 256 + kh * 128 + r] = pk[t];
}
// flag[panel] = 1 if a column of the panel holds a value that is not finite or has its values far below its maximum
__global__ __launch_bounds__(128) void i8_flag_panels_kernel(const unsigned* __restrict__ mx, const unsigned long long* __restrict__ stat, int N,
                                                              int* __restrict__ flag) {
  const int col = blockIdx.x * 128 + threadIdx.x;
  const unsigned long long q = col < N ? stat[col] : 0;
  const int bad = (col < N && mx[col] >= 0x7F800000u) || (unsigned)q < 16ull * (q >> 32);
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) flag[blockIdx.x] = any != 0;
}
struct ColumnWords { unsigned long long* stat; unsigned* mx; int* flag; };
size_t column_words(int64_t N) { return (size_t)(3 * N + (N + 127) / 128 + 1) / 2 * 2; }
ColumnWords column_words_at(unsigned* w, int N) { return ColumnWords{reinterpret_cast<unsigned long long*>(w), w + 2 * (size_t)N, reinterpret_cast<int*>(w + 3 * (size_t)N)}; }
template <int S, typename T>
void pack_columns(const T* X, int K, int N, int64_t ld, const ColumnWords& w, uint4* out, hipStream_t s) {
  const int np = (N + 127) / 128, nst = (K + 31) / 32;
  hipLaunchKernelGGL(i8_zero_kernel, dim3((3 * N + 255) / 256), dim3(256), 0, s, reinterpret_cast<unsigned*>(w.stat), 3 * N);      // stat and mx
  hipLaunchKernelGGL(i8_absbits_cols_kernel<T>, dim3((N + 255) / 256, (K + 127) / 128), dim3(256), 0, s, X, K, N, ld, w.mx);
  hipLaunchKernelGGL((i8_pack_rows_of_x_kernel<S, T>), dim3((unsigned)(((int64_t)nst * 2 * np * 128 + 255) / 256)), dim3(256), 0, s, X, K, N, ld, w.mx, w.stat, out, np, nst);
  hipLaunchKernelGGL(i8_flag_panels_kernel, dim3(np), dim3(128), 0, s, w.mx, w.stat, N, w.flag);
}
template <int S, typename T>
hipError_t i8_gram(const T* X, int64_t ldx, int d1, const T* Y, int64_t ldy, int m, int K, double* H64, double* G64, void* pack_x, void* pack_y,
                   unsigned* words, const int** flag_x, const int** flag_y, hipStream_t s) {
  uint4 *px = reinterpret_cast<uint4*>(pack_x), *py = reinterpret_cast<uint4*>(pack_y);
  const ColumnWords wx = column_words_at(words, d1);
  int log_slot = -1;
  gemm_log_open(d1, d1, K, 16 | 2 | 4 | 8, s, &log_slot);
  pack_columns<S>(X, K, d1, ldx, wx, px, s);
  I8Args a{};
  a.Ap = a.Bp = px; a.nstages = (K + 31) / 32; a.mxa = a.mxb = wx.mx; a.C64 = H64; a.ldc = d1; a.M = a.N = d1;
  a.tiles_m = a.tiles_n = (d1 + 127) / 128; a.lower_only = 1; a.skip_a = a.skip_b = wx.flag;
  const int nr = (a.tiles_m + 7) / 8;
  hipLaunchKernelGGL(i8_gemm_kernel<S>, dim3((unsigned)((nr * (nr + 1) / 2 + 7) / 8 * 8 * 64)), dim3(512), 0, s, a);
  gemm_log_close(log_slot, s);
  *flag_x = wx.flag;
  if (Y) {
    gemm_log_open(d1, m, K, 16 | 2, s, &log_slot);
    const ColumnWords wy = column_words_at(words + column_words(d1), m);
    pack_columns<S>(Y, K, m, ldy, wy, py, s);
    a.Bp = py; a.mxb = wy.mx; a.C64 = G64; a.ldc = m; a.N = m; a.tiles_n = (m + 127) / 128; a.lower_only = 0; a.skip_b = wy.flag;
    hipLaunchKernelGGL(i8_gemm_kernel<S>, dim3((unsigned)((nr * ((a.tiles_n + 7) / 8) + 7) / 8 * 8 * 64)), dim3(512), 0, s, a);
    gemm_log_close(log_slot, s);
    *flag_y = wy.flag;
  }
  return hipGetLastError();
}
}  // namespace
// rows that a packing buffer of `bytes` bytes takes at a time (a whole number of stages, at most 16384)
int64_t i8_gram_rows(size_t bytes, int x_bf16, int64_t cols) {
  const int64_t per_stage = (int64_t)(x_bf16 ? I8_S_BF16 : I8_S) * 256 * 16 * ((cols + 127) / 128);
  return std::min<int64_t>(16384, (int64_t)bytes / per_stage * 32);
}
size_t i8_gram_word_bytes(int64_t d1, int64_t m) { return (column_words(d1) + column_words(m)) * 4; }
hipError_t launch_i8_gram(const void* X, int x_bf16, int64_t ldx, int d1, const void* Y, int64_t ldy, int m, int K, double* H64, double* G64,
                          void* pack_x, void* pack_y, unsigned* words, const int** flag_x, const int** flag_y, hipStream_t s) {
  if (K <= 0) return hipErrorInvalidValue;
  if (K > 16384 || (reinterpret_cast<uintptr_t>(pack_x) & 15) || (Y && (reinterpret_cast<uintptr_t>(pack_y) & 15)) || (reinterpret_cast<uintptr_t>(words) & 7)) return hipErrorInvalidValue;
  if (x_bf16) return i8_gram<I8_S_BF16>(reinterpret_cast<const uint16_t*>(X), ldx, d1, reinterpret_cast<const uint16_t*>(Y), ldy, m, K, H64, G64, pack_x, pack_y, words, flag_x, flag_y, s);
  return i8_gram<I8_S>(reinterpret_cast<const float*>(X), ldx, d1, reinterpret_cast<const float*>(Y), ldy, m, K, H64, G64, pack_x, pack_y, words, flag_x, flag_y, s);
}

}  // namespace osscar
