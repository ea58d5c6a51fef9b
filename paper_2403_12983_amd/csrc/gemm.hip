// General matrix product on the gfx950 matrix cores with float32 storage and float64 accumulation.
//
//   C = alpha * A * op(B) + beta * Cin  (+ diag_add on the main diagonal)
//
// Used wherever the solver needs a result that is accurate to float32 rounding of the exact value:
// G = H W, the Newton-Schulz refinement of the inverse, B = P G_K with a float64 residual step, the
// candidate-side products V = P H_{K,Kc}, S = H_cc - H_cK V, R = G_c - H_cK B, and the block sweeps of
// the inverse.  Products of two float32 numbers are exact in float64, so the only rounding is the final
// conversion of each output element.
//
// Tiling: one workgroup of 256 threads (4 wave64 in a 2 x 2 grid) owns a 128 x 128 tile of C; each wave
// owns 64 x 64 as 4 x 4 v_mfma_f64_16x16x4_f64 tiles (64 float64 accumulators per lane).  A and B tiles
// of depth 16 are staged through LDS in k-major order ([k][row]) so that the 16 lanes of an MFMA operand
// column read consecutive LDS words.  Global loads for the next k-tile are issued before the MFMAs of
// the current one (register double buffering).
#include "internal.h"
#include <vector>

namespace osscar {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 16, LDT = BM + 4;

// Workgroup barrier that waits for this wave's LDS traffic only.  __syncthreads() also waits until every global load and
// store of the wave has completed, which in an epilogue that stages through LDS pass by pass makes each pass wait for the
// previous pass's stores to reach memory.  Only for hazards on LDS data.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

struct Tile8 { float v[8]; };

// 8 consecutive floats of a row starting at column c0 (element stride 1), zero beyond `ncols`.
__device__ __forceinline__ Tile8 load8(const float* __restrict__ row, int c0, int ncols, bool vec) {
  Tile8 t;
  if (row == nullptr) {
#pragma unroll
    for (int i = 0; i < 8; i++) t.v[i] = 0.f;
    return t;
  }
  if (vec && c0 + 8 <= ncols) {
    float4 a = *reinterpret_cast<const float4*>(row + c0);
    float4 b = *reinterpret_cast<const float4*>(row + c0 + 4);
    t.v[0] = a.x; t.v[1] = a.y; t.v[2] = a.z; t.v[3] = a.w;
    t.v[4] = b.x; t.v[5] = b.y; t.v[6] = b.z; t.v[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < 8; i++) t.v[i] = (c0 + i < ncols) ? row[c0 + i] : 0.f;
  }
  return t;
}

// Block -> tile.  Workgroups go to the 8 XCDs in turn (block index modulo 8), each with its own L2; two workgroups fit a
// CU, so 64 run together per XCD.  The tile grid is cut into 8 x 8 super-blocks, super-block b goes to XCD b % 8 and
// the 64 workgroups an XCD runs together are the 64 tiles of one super-block: they share 8 row panels of A and 8
// column panels of B in that L2.  Padding tiles return at once.  lower_only products take the super-blocks on or below
// the diagonal.
constexpr int SB = 8;
__device__ __forceinline__ bool tile_of_block(const GemmArgs& g, int& tile_m, int& tile_n) {
  if (g.lower_only) {
    // the super-blocks on or below the diagonal, row by row: sb = R (R + 1) / 2 + C, C <= R; in a diagonal super-block the
    // tiles above the diagonal return at once
    const int tm = (g.M + BM - 1) / BM, nr = (tm + SB - 1) / SB;
    const int b = blockIdx.x, xcd = b & 7, slot = b >> 3;
    const int sb = (slot / (SB * SB)) * 8 + xcd, within = slot % (SB * SB);
    if (sb >= nr * (nr + 1) / 2) return false;
    int r = (int)((sqrtf(8.f * (float)sb + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= sb) r++;
    while (r * (r + 1) / 2 > sb) r--;
    tile_m = r * SB + within / SB;
    tile_n = (sb - r * (r + 1) / 2) * SB + within % SB;
    return tile_m < tm && tile_n <= tile_m;
  }
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  const int nsb_c = (tn + SB - 1) / SB, nsb = ((tm + SB - 1) / SB) * nsb_c;
  const int b = blockIdx.x, xcd = b & 7, slot = b >> 3;
  const int sb = (slot / (SB * SB)) * 8 + xcd, within = slot % (SB * SB);
  if (sb >= nsb) return false;
  tile_m = (sb / nsb_c) * SB + within / SB;
  tile_n = (sb % nsb_c) * SB + within % SB;
  if (tile_m >= tm || tile_n >= tn) return false;
  return true;
}
static int grid_blocks(const GemmArgs& a) {
  const int tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
  if (a.lower_only) {
    const int nr = (tm + SB - 1) / SB;
    return (nr * (nr + 1) / 2 + 7) / 8 * 8 * SB * SB;
  }
  const int nsb = ((tm + SB - 1) / SB) * ((tn + SB - 1) / SB);
  return (nsb + 7) / 8 * 8 * SB * SB;
}

template <typename OutT>
__global__ __launch_bounds__(256, 2) void gemm_f64acc_kernel(GemmArgs g, int vecA, int vecB, int vecC) {
  // A and B stages; after the main loop the same memory stages the output tile (4 waves x 16 x 66 doubles)
  __shared__ __attribute__((aligned(16))) float smem[2 * 2 * BK * LDT];
  float (*As)[BK][LDT] = reinterpret_cast<float (*)[BK][LDT]>(smem);
  float (*Bs)[BK][LDT] = reinterpret_cast<float (*)[BK][LDT]>(smem + 2 * BK * LDT);

  int tile_m, tile_n;
  if (!tile_of_block(g, tile_m, tile_n)) return;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // global -> register staging assignments
  const int a_row = tid >> 1, a_k = (tid & 1) * 8;          // A tile: 128 rows x 16 k
  const int bt_row = tid >> 1, bt_k = (tid & 1) * 8;        // B^T given (N x K): 128 n-rows x 16 k
  const int b_k = tid >> 4, b_n = (tid & 15) * 8;           // B tile: 16 k x 128 n

  const float* a_ptr = (m0 + a_row < g.M) ? g.A + (int64_t)(m0 + a_row) * g.lda : nullptr;
  const float* bt_ptr = (g.trans_b && n0 + bt_row < g.N) ? g.B + (int64_t)(n0 + bt_row) * g.ldb : nullptr;

  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = d4{0, 0, 0, 0};

  const int ktiles = (g.K + BK - 1) / BK;
  Tile8 ra, rb;
  auto gload = [&](int kt) {
    int k0 = kt * BK;
    ra = load8(a_ptr, k0 + a_k, g.K, vecA);
    if (g.trans_b) {
      rb = load8(bt_ptr, k0 + bt_k, g.K, vecB);
    } else {
      const float* bp = (k0 + b_k < g.K) ? g.B + (int64_t)(k0 + b_k) * g.ldb : nullptr;
      rb = load8(bp, n0 + b_n, g.N, vecB);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 8; i++) As[buf][a_k + i][a_row] = ra.v[i];
    if (g.trans_b) {
#pragma unroll
      for (int i = 0; i < 8; i++) Bs[buf][bt_k + i][bt_row] = rb.v[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; i++) Bs[buf][b_k][b_n + i] = rb.v[i];
    }
  };

  if (ktiles > 0) { gload(0); sstore(0); }
  __syncthreads();
  for (int kt = 0; kt < ktiles; kt++) {
    int buf = kt & 1;
    if (kt + 1 < ktiles) gload(kt + 1);
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      int k = kk * 4 + (lane >> 4);
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; i++) a[i] = (double)As[buf][k][wm * 64 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; j++) b[j] = (double)Bs[buf][k][wn * 64 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < ktiles) sstore(buf ^ 1);
    __syncthreads();
  }

  // epilogue: lane holds D[4*r + lane/16][lane%16] of each 16 x 16 tile
  OutT* C = reinterpret_cast<OutT*>(g.C);
  const OutT* Cin = reinterpret_cast<const OutT*>(g.Cin);
  const bool use_cin = (Cin != nullptr && g.beta != 0.0);
  if (sizeof(OutT) == 4 && vecC) {
    // float output: each wave stages 16 x 64 of its tile in LDS and writes rows as float4 (256 contiguous bytes)
    constexpr int SLD = 66;
    double* st = reinterpret_cast<double*>(smem) + wave * 16 * SLD;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) st[(4 * r + (lane >> 4)) * SLD + j * 16 + (lane & 15)] = g.alpha * acc[i][j][r];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int lr = (lane >> 4) + 4 * k, lc = (lane & 15) * 4;
        const int row = m0 + wm * 64 + i * 16 + lr;
        const int col = n0 + wn * 64 + lc;
        if (row < g.M && col < g.N) {
          double v[4];
#pragma unroll
          for (int e = 0; e < 4; e++) v[e] = st[lr * SLD + lc + e];
          if (col + 3 < g.N) {
            if (use_cin) {
              const float4 ci = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(Cin) + (int64_t)row * g.ldcin + col);
              v[0] += g.beta * ci.x; v[1] += g.beta * ci.y; v[2] += g.beta * ci.z; v[3] += g.beta * ci.w;
            }
#pragma unroll
            for (int e = 0; e < 4; e++) if (row == col + e) v[e] += g.diag_add;
            float4 o = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + (int64_t)row * g.ldc + col) = o;
          } else {
            for (int e = 0; e < 4 && col + e < g.N; e++) {
              double x = v[e];
              if (use_cin) x += g.beta * (double)Cin[(int64_t)row * g.ldcin + col + e];
              if (row == col + e) x += g.diag_add;
              C[(int64_t)row * g.ldc + col + e] = (OutT)x;
            }
          }
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        int row = m0 + wm * 64 + i * 16 + 4 * r + (lane >> 4);
        int col = n0 + wn * 64 + j * 16 + (lane & 15);
        if (row < g.M && col < g.N) {
          double v = g.alpha * acc[i][j][r];
          if (use_cin) v += g.beta * (double)Cin[(int64_t)row * g.ldcin + col];
          if (row == col) v += g.diag_add;
          C[(int64_t)row * g.ldc + col] = (OutT)v;
        }
      }
}

// float32-accumulating variant (v_mfma_f32_32x32x2_f32, twice the rate of the float64 matrix path) for products whose
// result is added to float32 data anyway: the rank-64 sweeps of the inverse (refined afterwards) and the flushes of
// the delayed-update search.  Same tiling; each wave owns 64 x 64 as 2 x 2 tiles of 32 x 32.  float output only.
typedef float f16v __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256, 2) void gemm_f32acc_kernel(GemmArgs g, int vecA, int vecB, int vecC) {
  __shared__ __attribute__((aligned(16))) float smem[2 * 2 * BK * LDT];
  float (*As)[BK][LDT] = reinterpret_cast<float (*)[BK][LDT]>(smem);
  float (*Bs)[BK][LDT] = reinterpret_cast<float (*)[BK][LDT]>(smem + 2 * BK * LDT);
  int tile_m, tile_n;
  if (!tile_of_block(g, tile_m, tile_n)) return;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int a_row = tid >> 1, a_k = (tid & 1) * 8;
  const int bt_row = tid >> 1, bt_k = (tid & 1) * 8;
  const int b_k = tid >> 4, b_n = (tid & 15) * 8;
  const float* a_ptr = (m0 + a_row < g.M) ? g.A + (int64_t)(m0 + a_row) * g.lda : nullptr;
  const float* bt_ptr = (g.trans_b && n0 + bt_row < g.N) ? g.B + (int64_t)(n0 + bt_row) * g.ldb : nullptr;
  f16v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;
  const int kt_begin = 0;
  const int ktiles = (g.K + BK - 1) / BK;
  Tile8 ra, rb;
  auto gload = [&](int kt) {
    int k0 = kt * BK;
    ra = load8(a_ptr, k0 + a_k, g.K, vecA);
    if (g.trans_b) {
      rb = load8(bt_ptr, k0 + bt_k, g.K, vecB);
    } else {
      const float* bp = (k0 + b_k < g.K) ? g.B + (int64_t)(k0 + b_k) * g.ldb : nullptr;
      rb = load8(bp, n0 + b_n, g.N, vecB);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 8; i++) As[buf][a_k + i][a_row] = ra.v[i];
    if (g.trans_b) {
#pragma unroll
      for (int i = 0; i < 8; i++) Bs[buf][bt_k + i][bt_row] = rb.v[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; i++) Bs[buf][b_k][b_n + i] = rb.v[i];
    }
  };
  if (ktiles > kt_begin) { gload(kt_begin); sstore(kt_begin & 1); }
  __syncthreads();
  for (int kt = kt_begin; kt < ktiles; kt++) {
    int buf = kt & 1;
    if (kt + 1 < ktiles) gload(kt + 1);
#pragma unroll
    for (int kk = 0; kk < BK / 2; kk++) {
      const int k = kk * 2 + (lane >> 5);
      float a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; i++) a[i] = As[buf][k][wm * 64 + i * 32 + (lane & 31)];
#pragma unroll
      for (int j = 0; j < 2; j++) b[j] = Bs[buf][k][wn * 64 + j * 32 + (lane & 31)];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < ktiles) sstore(buf ^ 1);
    __syncthreads();
  }
  // epilogue: lane holds rows (r/4)*8 + (lane/32)*4 + r%4, column lane%32 of each 32 x 32 tile; staged per 32 rows
  float* C = reinterpret_cast<float*>(g.C);
  const float* Cin = g.Cin;
  const bool use_cin = (Cin != nullptr && g.beta != 0.0);
  const float alpha = (float)g.alpha, beta = (float)g.beta, dadd = (float)g.diag_add;
  constexpr int SLD = 68;
  float* st = smem + wave * 32 * SLD;          // 4 waves x 32 x 68 floats = 34816 bytes > smem: stage 16 rows at a time
  // This thread's Cin values are all requested before the first staging pass, and the passes are separated by barriers
  // that wait for LDS only: the loads' latency is paid once and no pass waits for the stores of the one before
  // (measured per workgroup on the rank-128 update of a 28672^2 triangle: epilogue 22.7 us, as long as the main loop,
  // 5.3 us of it in each of the four passes between its barriers).
  float4 cpre[2][2][4];
  const bool pre = use_cin && vecC;
  auto load_cin = [&](int i) {                   // the 32 rows i of this wave's 64: requested while the rows before them are
#pragma unroll                                   // still being staged, when the accumulators they replace are no longer live
    for (int half = 0; half < 2; half++)
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int row = m0 + wm * 64 + i * 32 + half * 16 + (lane >> 4) + 4 * k, col = n0 + wn * 64 + (lane & 15) * 4;
        cpre[i][half][k] = (row < g.M && col + 3 < g.N) ? *reinterpret_cast<const float4*>(Cin + (int64_t)row * g.ldcin + col)
                                                        : float4{0.f, 0.f, 0.f, 0.f};
      }
  };
  if (pre) load_cin(0);
#pragma unroll
  for (int i = 0; i < 2; i++) {
#pragma unroll
    for (int half = 0; half < 2; half++) {       // rows (r/4)*8 + ... with r/4 in {2*half, 2*half+1}
      lds_barrier();
      float* sth = smem + wave * 16 * SLD;
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int rq = 0; rq < 2; rq++)
#pragma unroll
          for (int r3 = 0; r3 < 4; r3++) {
            const int r = (2 * half + rq) * 4 + r3;
            sth[(rq * 8 + (lane >> 5) * 4 + r3) * SLD + j * 32 + (lane & 31)] = alpha * acc[i][j][r];
          }
      lds_barrier();
      if (pre && i == 0 && half == 1) load_cin(1);
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int lr = (lane >> 4) + 4 * k, lc = (lane & 15) * 4;     // 16 staged rows x 64 columns
        const int row = m0 + wm * 64 + i * 32 + half * 16 + lr;
        const int col = n0 + wn * 64 + lc;
        if (row < g.M && col < g.N) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; e++) v[e] = sth[lr * SLD + lc + e];
          if (vecC && col + 3 < g.N) {
            if (use_cin) {
              const float4 ci = cpre[i][half][k];
              v[0] += beta * ci.x; v[1] += beta * ci.y; v[2] += beta * ci.z; v[3] += beta * ci.w;
            }
#pragma unroll
            for (int e = 0; e < 4; e++) if (row == col + e) v[e] += dadd;
            *reinterpret_cast<float4*>(C + (int64_t)row * g.ldc + col) = float4{v[0], v[1], v[2], v[3]};
          } else {
            for (int e = 0; e < 4 && col + e < g.N; e++) {
              float x = v[e];
              if (use_cin) x += beta * Cin[(int64_t)row * g.ldcin + col + e];
              if (row == col + e) x += dadd;
              C[(int64_t)row * g.ldc + col + e] = x;
            }
          }
        }
      }
    }
  }
  (void)st;
}

// Optional log of every launch (shape, variant, duration by a pair of events on the launch's stream): a diagnostic that
// bench.py switches on for one untimed layer to report the time-weighted matrix-core rate over all launches.
namespace {
struct GemmLogEntry { int M, N, K, kind; hipEvent_t a, b; };
std::vector<GemmLogEntry> g_log;
bool g_log_on = false;
constexpr size_t GEMM_LOG_CAP = 16384;
}  // namespace
void gemm_log_enable(int on) {
  for (auto& e : g_log) { hipEventDestroy(e.a); hipEventDestroy(e.b); }
  g_log.clear();
  g_log_on = on != 0;
}
int gemm_log_read(double* out, int capacity) {
  int n = 0;
  for (auto& e : g_log) {
    if (n >= capacity) break;
    float ms = 0.f;
    if (hipEventSynchronize(e.b) != hipSuccess || hipEventElapsedTime(&ms, e.a, e.b) != hipSuccess) ms = -1.f;
    double* r = out + 5 * (size_t)n++;
    r[0] = e.M; r[1] = e.N; r[2] = e.K; r[3] = e.kind; r[4] = ms;
  }
  return n;
}

// the same log for launches made elsewhere (the int8 product): open records the first event, close the second
void gemm_log_open(int M, int N, int K, int kind, hipStream_t s, int* slot) {
  *slot = -1;
  if (!g_log_on || g_log.size() >= GEMM_LOG_CAP) return;
  GemmLogEntry e{M, N, K, kind, nullptr, nullptr};
  if (hipEventCreate(&e.a) != hipSuccess) return;
  if (hipEventCreate(&e.b) != hipSuccess) { hipEventDestroy(e.a); return; }
  hipEventRecord(e.a, s);
  g_log.push_back(e);
  *slot = (int)g_log.size() - 1;
}
void gemm_log_close(int slot, hipStream_t s) {
  if (slot >= 0 && slot < (int)g_log.size()) hipEventRecord(g_log[slot].b, s);
}

static hipError_t launch_gemm_impl(const GemmArgs& a, hipStream_t s);
hipError_t launch_gemm_f64acc(const GemmArgs& a, hipStream_t s) {
  if (!g_log_on || g_log.size() >= GEMM_LOG_CAP || a.M <= 0 || a.N <= 0) return launch_gemm_impl(a, s);
  GemmLogEntry e{a.M, a.N, a.K, (a.acc_f32 ? 1 : 0) | (a.c_is_f64 ? 2 : 0) | (a.lower_only ? 4 : 0) | (a.trans_b ? 8 : 0), nullptr, nullptr};
  if (hipEventCreate(&e.a) != hipSuccess || hipEventCreate(&e.b) != hipSuccess) return launch_gemm_impl(a, s);
  hipEventRecord(e.a, s);
  const hipError_t r = launch_gemm_impl(a, s);
  hipEventRecord(e.b, s);
  g_log.push_back(e);
  return r;
}

// Which of the two float64-accumulating kernels.  The 128 x 128 one needs about four rounds of two workgroups per compute
// unit to show its rate and 16-byte loads of both operands: 4096^3 2.26 ms against 2.70 ms of the 64 x 64 one, 8192 x 2048 x
// 8192 4.38 against 5.39 ms (1024 tiles each), but 1536 x 2048 x 1536 (192 tiles) 0.43 against 0.23 ms, 5461 x 1365 x 5461 (473
// tiles, unaligned rows) 3.55 against 1.98 ms, and a lower triangle of 7000 (1540 tiles, padding tiles among them) 7.6 against 7.2 ms.
static bool big_tiles_pay(const GemmArgs& a, bool vec) {
  const int64_t tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
  return vec && (a.lower_only ? tm * (tm + 1) / 2 >= 3072 : tm * tn >= 768);
}

static hipError_t launch_gemm_impl(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  const int blocks = grid_blocks(a);
  int vecA = (a.lda % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.A) & 15) == 0);
  int vecB = (a.ldb % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.B) & 15) == 0);
  int vecC = (!a.c_is_f64) && (a.ldc % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.C) & 15) == 0) &&
             (a.Cin == nullptr || ((a.ldcin % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.Cin) & 15) == 0)));
  if (a.acc_f32 && a.c_is_f64) return hipErrorInvalidValue;      // float32 accumulation has float32 output only
  // (a product that may accumulate in float32 takes it too: 1499 x 1003 x 1499 in 0.13 ms against 0.37 ms of 96 large tiles)
  if (!big_tiles_pay(a, vecA && vecB)) {
    Gemm64 q{};
    q.M = a.M; q.N = a.N; q.K = a.K; q.a_kind = OPK_ROW_F32; q.b_kind = a.trans_b ? OPK_ROW_F32 : OPK_K_F32; q.lower = a.lower_only;
    q.A = a.A; q.lda = a.lda; q.B = a.B; q.ldb = a.ldb; q.Cin = a.Cin; q.ldcin = a.ldcin; q.C = a.C; q.ldc = a.ldc; q.c_is_f64 = a.c_is_f64;
    q.alpha = a.alpha; q.beta = a.beta; q.diag_add = a.diag_add; q.ws = a.ws; q.ws_bytes = a.ws_bytes;
    return launch_gemm64(q, s);
  }
  if (a.acc_f32)
    hipLaunchKernelGGL(gemm_f32acc_kernel, dim3(blocks), dim3(256), 0, s, a, vecA, vecB, vecC);
  else if (a.c_is_f64)
    hipLaunchKernelGGL(gemm_f64acc_kernel<double>, dim3(blocks), dim3(256), 0, s, a, vecA, vecB, 0);
  else
    hipLaunchKernelGGL(gemm_f64acc_kernel<float>, dim3(blocks), dim3(256), 0, s, a, vecA, vecB, vecC);
  return hipGetLastError();
}

}  // namespace osscar
