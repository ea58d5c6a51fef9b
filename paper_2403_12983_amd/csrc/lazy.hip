// Delayed-update form of the local search for groups of one row (q = 1).
//
// The eager search applies every swap as a rank-2 pass over the whole tableau (N, Z): O(d1 (d1 + m)) bytes
// per swap.  Here the tableau in HBM is left at a BASE state (N0, Z0) and the swaps since then are kept as
// the set T of indices swept so far.  By the block form of the sweep operator, with C0 = N0[:, T],
// M = N0[T, T] and J = diag(-1 on the pivots that LEFT the kept set, +1 elsewhere),
//     N_cur[i, l] = N0[i, l] - C0[i, :] M^-1 C0[l, :]^T                (i, l outside T)
//     N_cur[T, l] = J M^-1 C0[l, :]^T,    N_cur[T, T] = -J M^-1 J
//     Z_cur[i, :] = Z0[i, :] - C0[i, :] ZT,   Z_cur[T, :] = J ZT,       ZT = M^-1 Z0[T, :]
// so one iteration needs only two columns of N_cur and the inner products of two rows of Z_cur, the diagonal
// and the squared row norms of Z_cur for the scores of eq. (impact) -- both updated incrementally, the
// norms through w = Z0 [y1 y2] -- and a bordering update of M^-1.
// w without a pass over Z0: y1, y2 are combinations of the current rows g, j of Z, and these of base rows:
//     Z0 z_g^T = Z0 Z0[g, :]^T - sum_r x_g[r] Z0 Z0[T_r, :]^T,     x_g = M^-1 C0[g, :]^T,
// so it is enough to know the products of Z0 with the base rows of g, j and of the pending pivots.  Which rows
// will be pivots before the next flush is predictable (in the largest layers the LAZY_NPICK_OUT cheapest removals and
// LAZY_NPICK_IN largest gains at flush time cover all but a few per thousand of them), so right after each flush one matrix
// product Zc Z0^T computes those products for these candidate rows (GbT); a pivot outside the candidates costs one read-only pass
// over Z0 for its column (kept in one of LAZY_NS spare slots), a launch of its own.  A layer of up to 11 blocks of 1024 rows takes all its
// picks from one of them if that is where they are; of more blocks each gives 1024 / blocks a side at most.  Every
// LAZY_TM/2 iterations the pending rank-tau correction is applied to N0 and Z0 by matrix products on the
// matrix cores.  The sequence of swaps is exactly that of the eager search (Proposition 4.1, Cases 1-3).
//
// A swap, or the removal of one row, is one launch (swap.hip); the rows that an iteration of the nested schedule prunes leave as one block
// pivot in two launches (below).
#include "internal.h"
#include "inverse16.h"
#include "lazy_device.h"
#include "wave.h"
#include <algorithm>

namespace osscar {


// ------------------------------------------------------------------------------------------------
// flush: apply the pending correction to N0, Z0 and empty T
// ------------------------------------------------------------------------------------------------
// pivot rows / columns of N0 and pivot rows of Z0.  Every entry is written by exactly one thread (the pending pivots are
// distinct), so the pivots are spread over blockIdx.y: FIX_SPB of them per thread.
constexpr int FIX_SPB = 8;
__global__ __launch_bounds__(256) void lazy_fix_kernel(LazyPtrs L, float* __restrict__ N0, int d1,
                                                        const SearchCtrl* __restrict__ ctrl) {
  const int l = blockIdx.x * 256 + threadIdx.x;
  if (l >= d1) return;
  const int tau = tau_all(ctrl);
  const int s0 = blockIdx.y * FIX_SPB, s1 = min(tau, s0 + FIX_SPB);
  if (s0 >= s1) return;
  const int pr = L.pos[l];
  if (pr < 0) {
    const float* El = L.E + (int64_t)l * LAZY_TM;
    for (int s = s0; s < s1; s++) {
      const int t = L.Tidx[s];
      const float v = L.Jsg[s] * El[s];
      if (l < t) N0[(int64_t)t * d1 + l] = v; else N0[(int64_t)l * d1 + t] = v;
    }
  } else {
    for (int s = s0; s < s1; s++) {
      const int t = L.Tidx[s];
      if (l >= t) N0[(int64_t)l * d1 + t] = (float)(-(double)L.Jsg[pr] * (double)L.Jsg[s] * L.Minv[pr * LAZY_TM + s]);
    }
  }
}
__global__ __launch_bounds__(256) void lazy_fix_z_kernel(LazyPtrs L, float* __restrict__ Z0, int m,
                                                          const SearchCtrl* __restrict__ ctrl) {
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= m) return;
  const int tau = tau_all(ctrl);
  const int s0 = blockIdx.y * FIX_SPB, s1 = min(tau, s0 + FIX_SPB);
  for (int s = s0; s < s1; s++) Z0[(int64_t)L.Tidx[s] * m + col] = (float)((double)L.Jsg[s] * L.ZT[(int64_t)s * m + col]);
}
__global__ __launch_bounds__(256) void lazy_reset_kernel(LazyPtrs L, SearchCtrl* ctrl) { empty_pending(L, ctrl, 256); }

// ------------------------------------------------------------------------------------------------
// candidate rows and their products with Z0 (after every flush)
// ------------------------------------------------------------------------------------------------
// ascending bitonic sort of 1024 (key, index) pairs, a thread each; equal keys: lower index first.  Exchanges at a distance below 64 stay
// inside a wave and go by shuffles, only the ten wider ones through shared memory (all through shared memory: 16 us; so: 6).
__device__ __forceinline__ void bitonic1024(double& key, int& idx, double* lk, int* li, int tid) {
  for (int k = 2; k <= 1024; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      double b;
      int ib;
      if (j >= 64) {
        __syncthreads();
        lk[tid] = key; li[tid] = idx;
        __syncthreads();
        b = lk[tid ^ j]; ib = li[tid ^ j];
      } else {
        b = __shfl_xor(key, j, 64); ib = __shfl_xor(idx, j, 64);
      }
      const bool after = (key > b) || (key == b && idx > ib);                     // this one comes after the other
      const bool low = (tid & j) == 0, up = (tid & k) == 0;
      if (after == (low == up) && !(key == b && idx == ib)) { key = b; idx = ib; }
    }
}

// per block of 1024 groups: the `per_block` cheapest removals among kept rows (blockIdx.y = 0) and the `per_block` largest gains
// among the others (1)
__global__ __launch_bounds__(1024) void cand_local_kernel(LazyPtrs L, int p, const int32_t* __restrict__ kept,
                                                           const double* __restrict__ score, int per_block) {
  __shared__ double lk[1024];
  __shared__ int li[1024];
  const int tid = threadIdx.x, h = blockIdx.x * 1024 + tid, nblk = gridDim.x, side = blockIdx.y;
  const bool valid = (h < p) && ((kept[h] != 0) == (side == 0));
  double key = valid ? (side == 0 ? score[h] : -score[h]) : INFINITY;
  if (key != key) key = INFINITY;      // not picked (with a NaN the two lanes of an exchange would disagree, and one row would be there twice, another not at all)
  int idx = valid ? h : 0x7fffffff;
  bitonic1024(key, idx, lk, li, tid);
  if (tid < per_block) {
    L.lkey[(side * nblk + blockIdx.x) * per_block + tid] = key;
    L.lidx[(side * nblk + blockIdx.x) * per_block + tid] = idx;
  }
}

// merge of the per-block winners, a workgroup per side: n_k kept rows into slots [0, n_k), n_c others into [n_k, n_k + n_c);
// unused slots hold -1.
__global__ __launch_bounds__(1024) void cand_merge_kernel(LazyPtrs L, int nblk, int per_block, int n_k, int n_c) {
  __shared__ double lk[1024];
  __shared__ int li[1024];
  const int tid = threadIdx.x, total = nblk * per_block, side = blockIdx.x;
  const int cnt = side == 0 ? n_k : n_c, base = side == 0 ? 0 : n_k;
  double key = tid < total ? L.lkey[side * total + tid] : INFINITY;
  int idx = tid < total ? L.lidx[side * total + tid] : 0x7fffffff;
  if (nblk > 1) bitonic1024(key, idx, lk, li, tid);      // (one block's are sorted)
  if (tid < cnt) {
    const bool have = key < INFINITY;
    L.cand[base + tid] = have ? idx : -1;
    if (have) L.cslot[idx] = base + tid;
  }
  if (side == 0) {
    for (int s = n_k + n_c + tid; s < LAZY_NC + LAZY_NS; s += 1024) L.cand[s] = -1;
  }
}

// Zc[s, :] = Z0[cand[s], :] (zero for unused slots)
__global__ __launch_bounds__(256) void cand_gather_kernel(LazyPtrs L, const float* __restrict__ Z0, int m) {
  const int s = blockIdx.x, r = L.cand[s];
  float* dst = L.Zc + (int64_t)s * m;
  for (int c = threadIdx.x; c < m; c += 256) dst[c] = (r >= 0) ? Z0[(int64_t)r * m + c] : 0.f;
}

// ------------------------------------------------------------------------------------------------
// The look-ahead product GbT[s, i] = <Z0[cand[s], :], Z0[i, :]> on the bf16 matrix cores, bound by one read of Z0.
// Every float32 number is cut into three bf16 pieces (each the round-to-nearest bf16 of what the pieces before it leave;
// together 24 significand bits) and the six products of weight >= 2^-16 run as v_mfma_f32_32x32x16_bf16: products of bf16
// numbers are exact in float32, the sums inside the matrix cores restart every 1024 columns (added, round to nearest,
// to a second float32 set), and every element of GbT is written once by the one wave that owns it (no atomics: the
// result does not depend on scheduling).  The candidate rows are cut and laid out in operand order once per flush
// (la_pack_kernel, a few MB that stay in L2); the rows of Z0 are cut in registers, each lane taking 8 consecutive
// columns of one row from the tile in shared memory, which is the operand layout as it stands.
//   one workgroup = 128 rows of Z0 x 128 candidates; wave w owns rows 32 w .. 32 w + 31 as four 32 x 32 tiles.
// ------------------------------------------------------------------------------------------------
typedef float la_f16v __attribute__((ext_vector_type(16)));
typedef __bf16 la_bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t la_u4 __attribute__((ext_vector_type(4)));      // (arrays of HIP's vector structs end in scratch memory)
typedef float la_f4 __attribute__((ext_vector_type(4)));
constexpr int LA_STG = 32;                   // columns of Z per stage (two 16-deep matrix-core steps)
// A workgroup multiplies its rows of Z0 with one block of NC = 32 NT candidates (NT = 4, 5 or 6 tiles of 32 per wave);
// packets per stage and block: 3 pieces x 4 groups of 8 columns x NC candidates.

// v[0..8) -> three packets of 8 bf16 each, by v_cvt_pk_bf16_f32 (round to nearest; two numbers an instruction where the same in whole
// numbers took eight)
__device__ __forceinline__ void la_split3(const float* v, uint4& p1, uint4& p2, uint4& p3) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  uint32_t h1[4], h2[4], h3[4];
  auto cut = [](float& x, float& y) -> uint32_t {
    const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{x, y}), b2));
    x -= __uint_as_float(u << 16); y -= __uint_as_float(u & 0xFFFF0000u);
    return u;
  };
#pragma unroll
  for (int j = 0; j < 4; j++) {
    float x = v[2 * j], y = v[2 * j + 1];
    h1[j] = cut(x, y); h2[j] = cut(x, y); h3[j] = cut(x, y);
  }
  p1 = uint4{h1[0], h1[1], h1[2], h1[3]};
  p2 = uint4{h2[0], h2[1], h2[2], h2[3]};
  p3 = uint4{h3[0], h3[1], h3[2], h3[3]};
}

// ZcP[(sb * nstg + stage) * 12 nc + piece * 4 nc + kg * nc + s] = columns stage*32 + kg*8 .. +8 of candidate sb*nc + s, piece
// `piece` (zero for unused slots and beyond column m).  grid (nstg, number of blocks of nc candidates), 256 threads.
__global__ __launch_bounds__(256) void la_pack_kernel(LazyPtrs L, const float* __restrict__ Z0, int m, int nstg, int nc, uint4* __restrict__ ZcP) {
  const int stage = blockIdx.x, sb = blockIdx.y, tid = threadIdx.x;
  uint4* out = ZcP + ((int64_t)sb * nstg + stage) * 12 * nc;
  for (int pk = tid; pk < 4 * nc; pk += 256) {
    const int kg = pk / nc, sl = pk % nc;
    const int r = L.cand[sb * nc + sl], c0 = stage * LA_STG + kg * 8;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = 0.f;
    if (r >= 0 && c0 + 8 <= m) {
      const float4 a = *reinterpret_cast<const float4*>(Z0 + (int64_t)r * m + c0);
      const float4 b = *reinterpret_cast<const float4*>(Z0 + (int64_t)r * m + c0 + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
    uint4 p1, p2, p3;
    la_split3(v, p1, p2, p3);
    out[pk] = p1; out[4 * nc + pk] = p2; out[8 * nc + pk] = p3;
  }
}

// GbT[(sb * NC + s) * d1 + i] for i in [128 blockIdx.x, +128), s in [0, NC), sb = blockIdx.y, NC = 32 NT.  m % 8 == 0.
// Per stage of 32 columns the workgroup copies its 128 x 32 tile of Z0 (each row's 128 bytes by eight neighbouring lanes)
// and the candidates' packed pieces into shared memory; the next stage's loads are in flight while this one is
// multiplied.  Two workgroups share a compute unit.
constexpr int LA_ZLD = LA_STG + 4;           // row stride of the Z0 tile in shared memory (floats)
template <int NT>
__global__ __launch_bounds__(256, 2) void la_product_kernel(const uint4* __restrict__ ZcP, const float* __restrict__ Z0, int d1, int m,
                                                             int nstg, double* __restrict__ GbT) {
  constexpr int NC = 32 * NT, PK = 12 * NC, NLD = (PK + 255) / 256;      // candidates, packets per stage, loads per thread
  __shared__ uint4 lzc[PK];                                    // 6 KB per 32 candidates
  __shared__ __attribute__((aligned(16))) float lz0[128 * LA_ZLD];   // 18 KB
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sb = blockIdx.y;
  const int i0 = blockIdx.x * 128;
  // blockIdx.z: which part of the contraction (gridDim.z = 1, or 2 with the sums joined by atomic additions to a zeroed GbT:
  // two terms added to zero give the same bits in either order)
  const int st_begin = (int)blockIdx.z * ((nstg + (int)gridDim.z - 1) / (int)gridDim.z);
  const int st_end = min(nstg, st_begin + (nstg + (int)gridDim.z - 1) / (int)gridDim.z);
  const uint4* src = ZcP + (int64_t)sb * nstg * PK + tid;
  // global -> shared assignment of the Z0 tile: thread t takes 4 columns (t % 8) * 4 of rows t / 8 + 32 j, j < 4
  const int lr = tid >> 3, lk = (tid & 7) * 4;
  auto rowp = [&](int j) { const int row = i0 + lr + 32 * j; return Z0 + (int64_t)(row < d1 ? row : d1 - 1) * m + lk; };
  const float *zsrc0 = rowp(0), *zsrc1 = rowp(1), *zsrc2 = rowp(2), *zsrc3 = rowp(3);      // rows past the end: clamped, never stored
  la_f16v acc[NT], acc2[NT];
#pragma unroll
  for (int t = 0; t < NT; t++)
#pragma unroll
    for (int r = 0; r < 16; r++) { acc[t][r] = 0.f; acc2[t][r] = 0.f; }
  uint4 zc[NLD];
  float4 zt0, zt1, zt2, zt3;
  auto gload = [&](int stage_) {
    const uint4* p_ = src + (int64_t)stage_ * PK;
#pragma unroll
    for (int i = 0; i < NLD; i++) zc[i] = (tid + 256 * i < PK) ? p_[256 * i] : uint4{0u, 0u, 0u, 0u};
    const bool in_ = stage_ * LA_STG + lk < m;              /* m % 4 == 0: a float4 is inside or outside as a whole */
    const float4 z_ = float4{0.f, 0.f, 0.f, 0.f};
    zt0 = in_ ? *reinterpret_cast<const float4*>(zsrc0 + stage_ * LA_STG) : z_;
    zt1 = in_ ? *reinterpret_cast<const float4*>(zsrc1 + stage_ * LA_STG) : z_;
    zt2 = in_ ? *reinterpret_cast<const float4*>(zsrc2 + stage_ * LA_STG) : z_;
    zt3 = in_ ? *reinterpret_cast<const float4*>(zsrc3 + stage_ * LA_STG) : z_;
  };
  if (st_begin >= st_end) return;
  gload(st_begin);
  int since = 0;
  const float* myrow = lz0 + (wave * 32 + (lane & 31)) * LA_ZLD + (lane >> 5) * 8;
  for (int stage = st_begin; stage < st_end; stage++) {
    __syncthreads();                                           // the previous stage has been read by every wave
#pragma unroll
    for (int i = 0; i < NLD; i++)
      if (tid + 256 * i < PK) lzc[tid + 256 * i] = zc[i];
    *reinterpret_cast<float4*>(lz0 + lr * LA_ZLD + lk) = zt0;
    *reinterpret_cast<float4*>(lz0 + (lr + 32) * LA_ZLD + lk) = zt1;
    *reinterpret_cast<float4*>(lz0 + (lr + 64) * LA_ZLD + lk) = zt2;
    *reinterpret_cast<float4*>(lz0 + (lr + 96) * LA_ZLD + lk) = zt3;
    __syncthreads();
    if (stage + 1 < st_end) gload(stage + 1);
#pragma unroll
    for (int ks = 0; ks < LA_STG / 16; ks++) {
      const float4 v0 = *reinterpret_cast<const float4*>(myrow + ks * 16), v1 = *reinterpret_cast<const float4*>(myrow + ks * 16 + 4);
      const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
      uint4 b1, b2, b3;
      la_split3(v, b1, b2, b3);
      const la_bf8 f1 = *reinterpret_cast<const la_bf8*>(&b1), f2 = *reinterpret_cast<const la_bf8*>(&b2), f3 = *reinterpret_cast<const la_bf8*>(&b3);
      const int off = (ks * 2 + (lane >> 5)) * NC + (lane & 31);
#pragma unroll
      for (int t = 0; t < NT; t++) {
        uint4 q1 = lzc[off + t * 32], q2 = lzc[4 * NC + off + t * 32], q3 = lzc[8 * NC + off + t * 32];
        const la_bf8 a1 = *reinterpret_cast<la_bf8*>(&q1), a2 = *reinterpret_cast<la_bf8*>(&q2), a3 = *reinterpret_cast<la_bf8*>(&q3);
        // smallest terms first
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a3, f1, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, f2, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, f3, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, f1, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, f2, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, f1, acc[t], 0, 0, 0);
      }
    }
    if (++since == 1024 / LA_STG && stage + 1 < st_end) {     // the sums inside the matrix cores never span more than 1024 columns
      since = 0;
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) { acc2[t][r] += acc[t][r]; acc[t][r] = 0.f; }
    }
  }
  // C layout of the 32 x 32 tile: register r = rr*4 + r3 holds row rr*8 + (lane/32)*4 + r3 (a candidate), column lane%32 (a row of Z0)
  const int i_lane = i0 + wave * 32 + (lane & 31);
  if (i_lane < d1) {
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int sl = t * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        double* dst = GbT + (int64_t)(sb * NC + sl) * d1 + i_lane;
        const double v = (double)acc[t][r] + (double)acc2[t][r];
        if (gridDim.z == 1) *dst = v; else unsafeAtomicAdd(dst, v);
      }
  }
}

// The same for layers whose rows do not fill the chip in 128s: 64 rows per workgroup and eight waves, wave w: rows 32 (w & 1) .., the 16 columns
// (w >> 1) & 1 of every stage, candidate tiles of half w >> 2.  The two halves of a stage meet in shared memory at the end, in this order.
// Bound by the chain of a stage (shared memory, cutting,
// eighteen products, two barriers), whose loads are requested three stages ahead.  8192 x 2048: 63 us (128 workgroups of 128 rows: 72);
// 3000 x 1000, a whole flush: 0.15 ms (0.20).
template <int NT>
__global__ __launch_bounds__(512) void la_product_rows64_kernel(const uint4* __restrict__ ZcP, const float* __restrict__ Z0, int d1, int m,
                                                                 int nstg, double* __restrict__ GbT) {
  constexpr int NC = 32 * NT, PK = 12 * NC, NLD = (PK + 511) / 512, TT = (NT + 1) / 2;
  __shared__ __attribute__((aligned(16))) uint4 lds[PK + 64 * LA_ZLD / 4];
  static_assert(sizeof(lds) >= 4 * 16 * 64 * sizeof(double), "a round of the final sums");
  la_u4* lzc = reinterpret_cast<la_u4*>(lds);
  float* lz0 = reinterpret_cast<float*>(lds + PK);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sb = blockIdx.y;
  const int rg = wave & 1, ks = (wave >> 1) & 1, ch = wave >> 2, t0 = ch * TT;
  const int i0 = blockIdx.x * 64;
  const int per = (nstg + (int)gridDim.z - 1) / (int)gridDim.z, st_begin = (int)blockIdx.z * per, st_end = min(nstg, st_begin + per);
  if (st_begin >= st_end) return;
  const uint4* src = ZcP + (int64_t)sb * nstg * PK + tid;
  const int lr = tid >> 3, lk = (tid & 7) * 4, row = min(i0 + lr, d1 - 1);      // rows past the end: clamped, never stored
  const float* zsrc = Z0 + (int64_t)row * m + lk;
  la_f16v acc[TT], acc2[TT];
#pragma unroll
  for (int t = 0; t < TT; t++)
#pragma unroll
    for (int r = 0; r < 16; r++) { acc[t][r] = 0.f; acc2[t][r] = 0.f; }
  la_u4 zc[3][NLD];                                            // three stages requested ahead
  la_f4 zt[3];
  auto gload = [&](int stage_, la_u4 (&q)[NLD], la_f4& z) {
    const int stage = min(stage_, st_end - 1);                 // (past the end: the last one again, not used)
    const la_u4* p = reinterpret_cast<const la_u4*>(src) + (int64_t)stage * PK;
#pragma unroll
    for (int i = 0; i < NLD; i++) q[i] = p[tid + 512 * i < PK ? 512 * i : 0];
    // (columns past the end: the row's first ones, replaced where they are stored: replaced here they would be waited for here)
    z = *reinterpret_cast<const la_f4*>(zsrc + (stage * LA_STG + lk < m ? stage * LA_STG : -lk));
  };
  const float* myrow = lz0 + (rg * 32 + (lane & 31)) * LA_ZLD + (lane >> 5) * 8 + ks * 16;
  int since = 0;
  auto one = [&](int stage, la_u4 (&q)[NLD], la_f4& z) {
    __syncthreads();                                           // the previous stage has been read by every wave
#pragma unroll
    for (int i = 0; i < NLD; i++)
      if (tid + 512 * i < PK) lzc[tid + 512 * i] = q[i];
    const bool in = stage * LA_STG + lk < m;                   // m % 4 == 0: a float4 is inside or outside as a whole
    *reinterpret_cast<la_f4*>(lz0 + lr * LA_ZLD + lk) = la_f4{in ? z.x : 0.f, in ? z.y : 0.f, in ? z.z : 0.f, in ? z.w : 0.f};
    __syncthreads();
    gload(stage + 3, q, z);
    const float4 v0 = *reinterpret_cast<const float4*>(myrow), v1 = *reinterpret_cast<const float4*>(myrow + 4);
    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    uint4 b1, b2, b3;
    la_split3(v, b1, b2, b3);
    const la_bf8 f1 = *reinterpret_cast<const la_bf8*>(&b1), f2 = *reinterpret_cast<const la_bf8*>(&b2), f3 = *reinterpret_cast<const la_bf8*>(&b3);
    const int off = (ks * 2 + (lane >> 5)) * NC + (lane & 31);
    la_bf8 a1[TT], a2[TT], a3[TT];
#pragma unroll
    for (int t = 0; t < TT; t++) {                             // (of an odd number of tiles the last one twice: the second is not stored)
      const int tt = min(t0 + t, NT - 1) * 32;
      a1[t] = __builtin_bit_cast(la_bf8, lzc[off + tt]); a2[t] = __builtin_bit_cast(la_bf8, lzc[4 * NC + off + tt]); a3[t] = __builtin_bit_cast(la_bf8, lzc[8 * NC + off + tt]);
    }
    auto mul = [&](const la_bf8 (&a)[TT], const la_bf8& f) {
#pragma unroll
      for (int t = 0; t < TT; t++) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], f, acc[t], 0, 0, 0);
    };
    mul(a3, f1); mul(a2, f2); mul(a1, f3); mul(a2, f1); mul(a1, f2); mul(a1, f1);      // smallest terms first
    if (++since == 1024 / LA_STG && stage + 1 < st_end) {      // (512 columns of each half of the stages)
      since = 0;
#pragma unroll
      for (int t = 0; t < TT; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) { acc2[t][r] += acc[t][r]; acc[t][r] = 0.f; }
    }
  };
#pragma unroll
  for (int i = 0; i < 3; i++) gload(st_begin + i, zc[i], zt[i]);
  for (int stage = st_begin; stage < st_end; stage += 3) {
    one(stage, zc[0], zt[0]);
    if (stage + 1 < st_end) one(stage + 1, zc[1], zt[1]);
    if (stage + 2 < st_end) one(stage + 2, zc[2], zt[2]);
  }
  // C layout of the 32 x 32 tile: register r = rr*4 + r3 holds row rr*8 + (lane/32)*4 + r3 (a candidate), column lane%32 (a row of Z0)
  double* half = reinterpret_cast<double*>(lds) + (rg * 2 + ch) * 16 * 64 + lane;
  const int i_lane = i0 + rg * 32 + (lane & 31);
#pragma unroll
  for (int t = 0; t < TT; t++) {
    __syncthreads();
    if (ks == 1)
#pragma unroll
      for (int r = 0; r < 16; r++) half[r * 64] = (double)acc[t][r] + (double)acc2[t][r];
    __syncthreads();
    if (ks == 0 && t0 + t < NT && i_lane < d1)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int sl = (t0 + t) * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        double* dst = GbT + (int64_t)(sb * NC + sl) * d1 + i_lane;
        const double v = ((double)acc[t][r] + (double)acc2[t][r]) + half[r * 64];
        if (gridDim.z == 1) *dst = v; else unsafeAtomicAdd(dst, v);
      }
  }
}

// mode 0: LAZY_NPICK_OUT slots for kept rows, LAZY_NPICK_IN for the others; 1: LAZY_NC for kept rows (removal-only loops); 2: none
struct CandCounts { int n_k, n_c; };
static CandCounts cand_counts(int mode) {
  // Swap search: a cycle of 64 swaps takes 64 pivots from each side, and which rows they will be is known at flush time only
  // up to the changes the swaps themselves make to the scores.  With exactly 64 + 64 rows picked, 8 % of the leaving and 2 %
  // of the entering pivots of the 28672 x 7168 layer were not among them, and each such swap pays a pass over Z0 for the
  // missing products (0.155 ms: 70 ms over 5000 swaps).  With 88 + 72 it is 0.4 % and 0.2 % (80 + 80: 1.3 % and none;
  // 96 + 64: 0.2 % and 2 %), for a product that is a quarter longer.  256 picked rows (two blocks of the product) cost more
  // than they save.  The removal-only loops take all LAZY_NC rows: their block pivots cannot fetch a missing product.
  static_assert((LAZY_NPICK_OUT + LAZY_NPICK_IN) % 32 == 0 && LAZY_NPICK_OUT + LAZY_NPICK_IN <= LAZY_NC, "blocks of 32 candidates");
  return CandCounts{mode == 2 ? 0 : (mode == 1 ? LAZY_NC : LAZY_NPICK_OUT), mode == 0 ? LAZY_NPICK_IN : 0};
}
// the pick: reads the scores and the kept flags only (two sorts in one workgroup each: latency, no bandwidth)
static hipError_t launch_candidate_pick(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode) {
  const int nblk = (d.p + 1023) / 1024;               // <= 64 (d1 <= 65536)
  // A side's winners are merged by one workgroup of 1024.  Of few blocks every one gives as many as are picked in all: with 32 of each
  // a layer of 826 rows missed half of its pivots, and one of 2000 a seventh.
  const CandCounts cc = cand_counts(mode);
  const int per_block = std::min(std::max({cc.n_k, cc.n_c, 1}), 1024 / nblk);
  hipError_t e = hipMemsetAsync(L.cslot, 0xFF, (size_t)d.d1 * 4, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cand_local_kernel, dim3(nblk, 2), dim3(1024), 0, s, L, d.p, t.kept, t.score, per_block);
  hipLaunchKernelGGL(cand_merge_kernel, dim3(2), dim3(1024), 0, s, L, nblk, per_block, cc.n_k, cc.n_c);
  return hipGetLastError();
}
// the products of the picked rows with one another and with the (flushed) Z0
static hipError_t launch_candidate_products(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode) {
  const CandCounts cc = cand_counts(mode);
  const int n_k = cc.n_k, n_c = cc.n_c;
  if (mode == 2) return hipSuccess;
  const hipError_t ek = launch_cand_gram(d, t, L, n_k + n_c, s);
  if (ek != hipSuccess) return ek;
  // one block of 32 NT candidates per workgroup: 128 (and multiples of it, block by block), 160 or 192
  const int ncand = n_k + n_c;
  const int nt = (ncand % 128 == 0) ? 4 : ((ncand == 160) ? 5 : ((ncand == 192) ? 6 : 0));
  if (d.m % 8 == 0 && nt > 0) {
    const int nstg = (d.m + LA_STG - 1) / LA_STG, nc = 32 * nt, nsb = ncand / nc;
    hipLaunchKernelGGL(la_pack_kernel, dim3(nstg, nsb), dim3(256), 0, s, L, t.Z, d.m, nstg, nc, reinterpret_cast<uint4*>(L.ZcP));
    // One block of candidates: 224 workgroups for 28672 rows would leave compute units empty and each of them with one latency chain over
    // all of m; the contraction is then cut in two.  Below 200 workgroups of 128 rows: 64 rows each, cut in two where they are fewer than 256.
    const int wgs = (d.d1 + 127) / 128 * nsb;
    const bool small = wgs < 200;
    const int wgs64 = (d.d1 + 63) / 64 * nsb;
    const int ksplit = small ? (wgs64 < 256 && nstg >= 16 ? 2 : 1) : (wgs < 400 && nstg >= 64) ? 2 : 1;
    if (ksplit > 1) {
      const hipError_t ez = hipMemsetAsync(L.GbT, 0, (size_t)ncand * d.d1 * sizeof(double), s);
      if (ez != hipSuccess) return ez;
    }
    const dim3 grid(small ? (d.d1 + 63) / 64 : (d.d1 + 127) / 128, nsb, ksplit);
    const uint4* zcp = reinterpret_cast<const uint4*>(L.ZcP);
    if (small) {
      if (nt == 4) hipLaunchKernelGGL(la_product_rows64_kernel<4>, grid, dim3(512), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
      else if (nt == 5) hipLaunchKernelGGL(la_product_rows64_kernel<5>, grid, dim3(512), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
      else hipLaunchKernelGGL(la_product_rows64_kernel<6>, grid, dim3(512), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
    } else if (nt == 4) hipLaunchKernelGGL(la_product_kernel<4>, grid, dim3(256), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
    else if (nt == 5) hipLaunchKernelGGL(la_product_kernel<5>, grid, dim3(256), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
    else hipLaunchKernelGGL(la_product_kernel<6>, grid, dim3(256), 0, s, zcp, t.Z, d.d1, d.m, nstg, L.GbT);
    return hipGetLastError();
  }
  // other shapes: the general matrix-product kernel on the gathered rows
  hipLaunchKernelGGL(cand_gather_kernel, dim3(n_k + n_c), dim3(256), 0, s, L, t.Z, d.m);
  GemmArgs g{};                         // GbT[0 .. LAZY_NC) = Zc Z0^T, float64 accumulation and output
  g.M = n_k + n_c; g.N = d.d1; g.K = d.m; g.A = L.Zc; g.lda = d.m; g.B = t.Z; g.ldb = d.m; g.trans_b = 1;
  g.C = L.GbT; g.ldc = d.d1; g.alpha = 1.0; g.beta = 0.0; g.c_is_f64 = 1; g.ws = L.gemm_ws; g.ws_bytes = L.gemm_ws_bytes;
  return launch_gemm_f64acc(g, s);
}
// what the next iteration picks from: the removal lists of the removal-only loops, the records of the swaps
// (refresh: after a flush, with the second half of the score refresh and the pending set emptied in the same launch)
static hipError_t launch_picks(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode, bool refresh) {
  return mode == 1 ? launch_removal_lists(d, t, L, s, refresh) : launch_swap_records(d, t, L, s, refresh);
}

// ------------------------------------------------------------------------------------------------
// The two rank-LAZY_TM updates of a flush, C -= A B^T with A (M x 128) and B (N x 128): N0 -= E C0^T on the lower block
// triangle and Z0 -= C0 ZT.  Both are bound by the read and write of C once the product itself is cheap, so the three
// thin operands (E, C0, ZT: a few MB) are cut into three bf16 pieces once per flush and laid out in matrix-core operand
// order (rk_pack_*), and the six products of weight >= 2^-16 run as v_mfma_f32_32x32x16_bf16 (exact products, float32
// sums over the 128 terms): a sixth of the matrix-core time of the float32 instruction for the same accuracy.
// Layout of a packed operand: packet (piece, kg, row) = columns 8 kg .. 8 kg + 7 of `row`, at (piece * 16 + kg) * rpad + row.
// One workgroup per 128 x 128 tile of C (the Gram kernel's tile schedules), four quarters of the contraction through
// 48 KB of shared memory, two workgroups per compute unit so that one's read-modify-write of C overlaps the other's products.
// ------------------------------------------------------------------------------------------------
// X: rows x 128 row-major (ld = 128): thread = one packet
__global__ __launch_bounds__(256) void rk_pack_rows_kernel(const float* __restrict__ X, int rows, int rpad, uint4* __restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;          // (kg, row), row fastest
  if (idx >= 16 * rpad) return;
  const int kg = idx / rpad, row = idx % rpad;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; j++) v[j] = 0.f;
  if (row < rows) {
    const float4 a = *reinterpret_cast<const float4*>(X + (int64_t)row * LAZY_TM + kg * 8);
    const float4 b = *reinterpret_cast<const float4*>(X + (int64_t)row * LAZY_TM + kg * 8 + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  uint4 p1, p2, p3;
  la_split3(v, p1, p2, p3);
  out[(int64_t)kg * rpad + row] = p1;
  out[(int64_t)(16 + kg) * rpad + row] = p2;
  out[(int64_t)(32 + kg) * rpad + row] = p3;
}
// X: 128 x cols row-major (the contraction runs along the rows): packet (kg, c) = X[8 kg .. 8 kg + 7][c]
__global__ __launch_bounds__(256) void rk_pack_cols_kernel(const float* __restrict__ X, int cols, int cpad, uint4* __restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= 16 * cpad) return;
  const int kg = idx / cpad, c = idx % cpad;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; j++) v[j] = (c < cols) ? X[(int64_t)(kg * 8 + j) * cols + c] : 0.f;
  uint4 p1, p2, p3;
  la_split3(v, p1, p2, p3);
  out[(int64_t)kg * cpad + c] = p1;
  out[(int64_t)(16 + kg) * cpad + c] = p2;
  out[(int64_t)(32 + kg) * cpad + c] = p3;
}

// Sums of squares of the new values of a wave's 32 rows x 64 columns, one number per row, into out[row] (rows_left of them
// exist).  v0, v1: the two 32 x 32 tiles side by side in the matrix cores' result layout (register r = rr*4 + r3 holds row
// rr*8 + (lane/32)*4 + r3, column lane%32).  Squares and sums in float64; the 32 lanes of a half wave are added by
// data-parallel moves in a fixed order, and lanes 31 and 63 write.
__device__ __forceinline__ void rk_row_squares(const float* v0, const float* v1, double* __restrict__ out, int lane, int rows_left) {
#pragma unroll
  for (int r = 0; r < 16; r++) {
    double q = (double)v0[r] * (double)v0[r] + (double)v1[r] * (double)v1[r];
    q += dpp_get<0xb1, 0xf>(q);        // quad_perm [1, 0, 3, 2]
    q += dpp_get<0x4e, 0xf>(q);        // quad_perm [2, 3, 0, 1]
    q += dpp_get<0x124, 0xf>(q);       // row_ror:4
    q += dpp_get<0x128, 0xf>(q);       // row_ror:8
    q += dpp_get<0x142, 0xa>(q);       // row_bcast:15 into rows 1 and 3: lanes 16-31 and 48-63 hold their half wave's sum
    const int row = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
    if ((lane & 31) == 31 && row < rows_left) out[row] = q;
  }
}

__global__ __launch_bounds__(256, 2) void rk_update_kernel(const uint4* __restrict__ Apk, int apad, const uint4* __restrict__ Bpk, int bpad,
                                                            float* __restrict__ C, int64_t ldc, int M, int N,
                                                            const int2* __restrict__ tiles, double* __restrict__ rowsq) {
  __shared__ uint4 la[3 * 4 * 128], lb[3 * 4 * 128];          // 24 KB each: [piece][kg of this quarter][row]
  const int2 tile = tiles[blockIdx.x];
  if (tile.x < 0) return;
  const int i0 = tile.x * 128, j0 = tile.y * 128;
  if (i0 >= M || j0 >= N) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  la_f16v acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[a][b][r] = 0.f;
  // packet tid + 256 u of a quarter's 1536: piece = idx / 512, kg = (idx / 128) % 4, row = idx % 128
  uint4 ra0, ra1, ra2, ra3, ra4, ra5, rb0, rb1, rb2, rb3, rb4, rb5;
#define OSSCAR_RK_ADDR(P_, pad_, base_, u_, kq_) \
  ((P_) + (int64_t)((((tid + 256 * (u_)) >> 9) * 16 + (kq_) * 4 + (((tid + 256 * (u_)) >> 7) & 3))) * (pad_) + (base_) + ((tid + 256 * (u_)) & 127))
#define OSSCAR_RK_GLOAD(kq_)                                                                                       \
  {                                                                                                                \
    ra0 = *OSSCAR_RK_ADDR(Apk, apad, i0, 0, kq_); ra1 = *OSSCAR_RK_ADDR(Apk, apad, i0, 1, kq_);                    \
    ra2 = *OSSCAR_RK_ADDR(Apk, apad, i0, 2, kq_); ra3 = *OSSCAR_RK_ADDR(Apk, apad, i0, 3, kq_);                    \
    ra4 = *OSSCAR_RK_ADDR(Apk, apad, i0, 4, kq_); ra5 = *OSSCAR_RK_ADDR(Apk, apad, i0, 5, kq_);                    \
    rb0 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 0, kq_); rb1 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 1, kq_);                    \
    rb2 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 2, kq_); rb3 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 3, kq_);                    \
    rb4 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 4, kq_); rb5 = *OSSCAR_RK_ADDR(Bpk, bpad, j0, 5, kq_);                    \
  }
#define OSSCAR_RK_STAGE()                                                                                          \
  {                                                                                                                \
    __syncthreads();                                                                                               \
    la[tid] = ra0; la[tid + 256] = ra1; la[tid + 512] = ra2; la[tid + 768] = ra3; la[tid + 1024] = ra4; la[tid + 1280] = ra5; \
    lb[tid] = rb0; lb[tid + 256] = rb1; lb[tid + 512] = rb2; lb[tid + 768] = rb3; lb[tid + 1024] = rb4; lb[tid + 1280] = rb5; \
    __syncthreads();                                                                                               \
  }
// the six piece products of a quarter, smallest terms first
#define OSSCAR_RK_PRODUCTS()                                                                                       \
  _Pragma("unroll") for (int ks = 0; ks < 2; ks++) {                                                               \
    const int off = (ks * 2 + (lane >> 5)) * 128 + (lane & 31);                                                    \
    la_bf8 fa[2][3], fb[2][3];                                                                                     \
    _Pragma("unroll") for (int a = 0; a < 2; a++)                                                                  \
      _Pragma("unroll") for (int p = 0; p < 3; p++) { uint4 q = la[p * 512 + off + wm * 64 + a * 32]; fa[a][p] = *reinterpret_cast<la_bf8*>(&q); } \
    _Pragma("unroll") for (int b = 0; b < 2; b++)                                                                  \
      _Pragma("unroll") for (int p = 0; p < 3; p++) { uint4 q = lb[p * 512 + off + wn * 64 + b * 32]; fb[b][p] = *reinterpret_cast<la_bf8*>(&q); } \
    _Pragma("unroll") for (int a = 0; a < 2; a++)                                                                  \
      _Pragma("unroll") for (int b = 0; b < 2; b++) {                                                              \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][2], fb[b][0], acc[a][b], 0, 0, 0);               \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][0], fb[b][2], acc[a][b], 0, 0, 0);               \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][1], fb[b][1], acc[a][b], 0, 0, 0);               \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][1], fb[b][0], acc[a][b], 0, 0, 0);               \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][0], fb[b][1], acc[a][b], 0, 0, 0);               \
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a][0], fb[b][0], acc[a][b], 0, 0, 0);               \
      }                                                                                                            \
  }
  OSSCAR_RK_GLOAD(0);
#pragma unroll 1
  for (int kq = 0; kq < 3; kq++) {
    OSSCAR_RK_STAGE();
    OSSCAR_RK_GLOAD(kq + 1);
    OSSCAR_RK_PRODUCTS();
  }
  OSSCAR_RK_STAGE();
  // C layout of a 32 x 32 tile: register r = rr*4 + r3 holds row rr*8 + (lane/32)*4 + r3, column lane%32.
  // A whole tile's values of C are requested before the last quarter's products, in the registers the operand loads have
  // left free, so that their way from memory runs beside the matrix-core work instead of after it (requesting half of them
  // a quarter earlier changed nothing).
  float* cbase = C + (int64_t)(i0 + wm * 64 + (lane >> 5) * 4) * ldc + j0 + wn * 64 + (lane & 31);
  const bool whole = (i0 + 128 <= M && j0 + 128 <= N);
  float cv[2][2][16];
  if (whole) {
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float* pr = cbase + (int64_t)(a * 32 + (r >> 2) * 8 + (r & 3)) * ldc;
        cv[a][0][r] = pr[0]; cv[a][1][r] = pr[32];
      }
  }
  OSSCAR_RK_PRODUCTS();
#undef OSSCAR_RK_PRODUCTS
#undef OSSCAR_RK_STAGE
#undef OSSCAR_RK_GLOAD
#undef OSSCAR_RK_ADDR
  if (whole) {
#pragma unroll
    for (int a = 0; a < 2; a++) {
      float* ca = cbase + (int64_t)(a * 32) * ldc;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        float* pr = ca + (int64_t)((r >> 2) * 8 + (r & 3)) * ldc;
        cv[a][0][r] -= acc[a][0][r]; cv[a][1][r] -= acc[a][1][r];
        pr[0] = cv[a][0][r]; pr[32] = cv[a][1][r];
      }
      if (rowsq) rk_row_squares(cv[a][0], cv[a][1], rowsq + (int64_t)(tile.y * 2 + wn) * M + i0 + wm * 64 + a * 32, lane, M - (i0 + wm * 64 + a * 32));
    }
  } else {
#pragma unroll
    for (int a = 0; a < 2; a++) {
      float nv[2][16];
#pragma unroll
      for (int b = 0; b < 2; b++) {
        const int col = j0 + wn * 64 + b * 32 + (lane & 31);
        float cv[16];
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int row = i0 + wm * 64 + a * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
          cv[r] = (row < M && col < N) ? C[(int64_t)row * ldc + col] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int row = i0 + wm * 64 + a * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
          const bool in = row < M && col < N;
          nv[b][r] = in ? cv[r] - acc[a][b][r] : 0.f;
          if (in) C[(int64_t)row * ldc + col] = nv[b][r];
        }
      }
      if (rowsq) rk_row_squares(nv[0], nv[1], rowsq + (int64_t)(tile.y * 2 + wn) * M + i0 + wm * 64 + a * 32, lane, M - (i0 + wm * 64 + a * 32));
    }
  }
}

// E = C0 M^-1 of the flush (d1 x 128 times 128 x 128, float32 operands, float64 sums on v_mfma_f64_16x16x4_f64, float32
// result).  It stands at the head of the flush's longer chain, so what counts is its latency: a workgroup takes 32 rows (256 workgroups
// at 8192 rows) with all of M^-1 and its rows of C0 in shared memory, no barrier inside the contraction; every thread has its share of
// both requested at once.  M^-1 (rounded to float32 here, zero from tau on) is symmetric bit for bit, so its rows serve as the
// columns the product needs.  Wave w: rows 16 (w & 1) .. + 15, columns 32 (w >> 1) .. + 31.
// 20 us at 8192 rows beside Z0's update (as 128 workgroups of 64 rows 26), 60 us at 28672 either way.
typedef double te_d4 __attribute__((ext_vector_type(4)));
constexpr int TE_LD = LAZY_TM + 4;       // row stride in shared memory (floats): a quarter wave's 16 rows x 4 k fall on 32 banks twice
constexpr int TE_ROWS = 32;
__global__ __launch_bounds__(512) void thin_e_kernel(LazyPtrs L, int d1, const SearchCtrl* __restrict__ ctrl) {
  static_assert(LAZY_TM == 128, "four pairs of column tiles, thirty-two steps of four");
  extern __shared__ float te_lds[];      // [128 rows of M^-1 | 32 rows of C0][TE_LD]
  float* Ms = te_lds;
  float* As = te_lds + LAZY_TM * TE_LD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i0 = blockIdx.x * TE_ROWS;
  const float* C0R = L.C0R;
  const double* Mi = L.Minv;
  const int tau = tau_all(ctrl);
  float4 c[2];
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int idx = tid + 512 * u, r = min(i0 + (idx >> 5), d1 - 1);
    c[u] = *reinterpret_cast<const float4*>(C0R + (int64_t)r * LAZY_TM + (idx & 31) * 4);
  }
  double2 v[16];
#pragma unroll
  for (int u = 0; u < 16; u++) {
    const int idx = tid + 512 * u;
    v[u] = *reinterpret_cast<const double2*>(Mi + (idx >> 6) * LAZY_TM + (idx & 63) * 2);
  }
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int idx = tid + 512 * u;
    *reinterpret_cast<float4*>(As + (idx >> 5) * TE_LD + (idx & 31) * 4) = c[u];
  }
#pragma unroll
  for (int u = 0; u < 16; u++) {
    const int idx = tid + 512 * u, r = idx >> 6, k = (idx & 63) * 2;
    *reinterpret_cast<float2*>(Ms + r * TE_LD + k) = float2{r < tau && k < tau ? (float)v[u].x : 0.f, r < tau && k + 1 < tau ? (float)v[u].y : 0.f};
  }
  __syncthreads();
  te_d4 acc[2] = {te_d4{0.0, 0.0, 0.0, 0.0}, te_d4{0.0, 0.0, 0.0, 0.0}};
  const float* arow = As + ((wave & 1) * 16 + (lane & 15)) * TE_LD + (lane >> 4);
  const float* mrow = Ms + ((wave >> 1) * 32 + (lane & 15)) * TE_LD + (lane >> 4);
#pragma unroll 8
  for (int k0 = 0; k0 < LAZY_TM; k0 += 4) {
    const double a = (double)arow[k0];
#pragma unroll
    for (int ct = 0; ct < 2; ct++) acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)mrow[ct * 16 * TE_LD + k0], acc[ct], 0, 0, 0);
  }
  // lane holds D[4 r + lane/16][lane%16] of each 16 x 16 tile
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int row = i0 + (wave & 1) * 16 + 4 * r + (lane >> 4);
    if (row < d1) {
#pragma unroll
      for (int ct = 0; ct < 2; ct++) L.E[(int64_t)row * LAZY_TM + (wave >> 1) * 32 + ct * 16 + (lane & 15)] = (float)acc[ct][r];
    }
  }
}

// First half of the score refresh after a flush: gram[h] = |Z0[h, :]|^2 from the stretch sums that Z0's update left (added in
// a fixed order), dblk[h] = N0[h][h].  The pending pivots' rows were rewritten after the update (the fix): the trailing
// LAZY_TM workgroups take one of them each and sum its squares from Z0 itself (wave sums, then the four waves in order).
__global__ __launch_bounds__(256) void norms_from_stretches_kernel(LazyPtrs L, int d1, int m, int nstretch, int row_blocks,
                                                                    const float* __restrict__ N0, const float* __restrict__ Z0,
                                                                    double* __restrict__ gram, double* __restrict__ dblk,
                                                                    const SearchCtrl* __restrict__ ctrl) {
  if ((int)blockIdx.x < row_blocks) {
    const int h = blockIdx.x * 256 + threadIdx.x;
    if (h >= d1) return;
    dblk[h] = (double)N0[(int64_t)h * d1 + h];
    if (L.pos[h] >= 0) return;                     // a pending pivot: its row is summed below
    double v = 0;
    for (int p0 = 0; p0 < nstretch; p0 += 8) {     // eight loads in flight
      double q[8];
#pragma unroll
      for (int u = 0; u < 8; u++) q[u] = (p0 + u < nstretch) ? L.rowsq[(int64_t)(p0 + u) * d1 + h] : 0.0;
#pragma unroll
      for (int u = 0; u < 8; u++) v += q[u];
    }
    gram[h] = v;
    return;
  }
  __shared__ double red[4];
  const int sidx = blockIdx.x - row_blocks;
  if (sidx >= tau_all(ctrl)) return;
  const int h = L.Tidx[sidx];
  const float* z = Z0 + (int64_t)h * m;
  double v = 0;
  for (int c = threadIdx.x; c < m; c += 256) v += (double)z[c] * (double)z[c];
  v = wsum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) gram[h] = red[0] + red[1] + red[2] + red[3];
}

hipError_t launch_lazy_flush(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode,
                             const SideStream* side) {
  const int rb = (d.d1 + 255) / 256, mb = (d.m + 255) / 256;
  const bool two = side && side->stream;
  hipStream_t sn = two ? side->stream : s;          // stream of the N0 update
  hipError_t err;
  // With two streams the chains of N0 (pick of the candidates, E, its pieces, update, fix, diagonal) and of Z0 (ZT, pieces, update, fix,
  // the candidates' products) run side by side from the start; the events between them: the pieces of C0 are packed here, the
  // pick is done there, both matrices are final.  (With E, all pieces and the pick before or between them on this stream a flush
  // of 8192 x 2048 was 0.06 ms longer.)
  auto here_to_there = [&]() -> hipError_t {
    if (!two) return hipSuccess;
    const hipError_t e = hipEventRecord(side->fork, s);
    return e != hipSuccess ? e : hipStreamWaitEvent(sn, side->fork, 0);
  };
  if ((err = here_to_there()) != hipSuccess) return err;
  // the three thin operands in matrix-core order (C0's pieces serve both updates)
  const int dpad = (d.d1 + 127) / 128 * 128, mpad = (d.m + 127) / 128 * 128;
  uint4* Epk = reinterpret_cast<uint4*>(L.Epk); uint4* Cpk = reinterpret_cast<uint4*>(L.Cpk); uint4* Zpk = reinterpret_cast<uint4*>(L.Zpk);
  // Launches take the host as long as the small ones run, so each stream's first ones come before the other's later ones (with all of
  // N0's up to its update in front of the first of Z0's a flush was 20 us longer)
  hipLaunchKernelGGL(rk_pack_rows_kernel, dim3((16 * dpad + 255) / 256), dim3(256), 0, s, L.C0R, d.d1, dpad, Cpk);
  if (two) {
    // The candidates of the next cycle, from the scores as the swaps left them (the refresh below changes them in the last
    // digits only, and the choice of candidates decides what is computed ahead, not any result)
    if ((err = launch_candidate_pick(d, t, L, sn, mode)) != hipSuccess) return err;
    if ((err = hipEventRecord(side->join, sn)) != hipSuccess) return err;
    if ((err = hipEventRecord(side->fork, s)) != hipSuccess) return err;      // the pieces of C0
  }
  if ((err = launch_zt(d, t, L, s)) != hipSuccess) return err;
  hipLaunchKernelGGL(rk_pack_cols_kernel, dim3((16 * mpad + 255) / 256), dim3(256), 0, s, L.ZT32, d.m, mpad, Zpk);
  // Z0 -= C0 ZT
  // (with two streams the kernel also leaves the sums of squares of every row's 64-column stretches: the row norms of the
  // score refresh then come from these 25 MB instead of another pass over Z0)
  auto update_z = [&]() {
    hipLaunchKernelGGL(rk_update_kernel, dim3((unsigned)L.n_tiles_rect), dim3(256), 0, s, Cpk, dpad, Zpk, mpad, t.Z, (int64_t)d.m, d.d1, d.m,
                       L.tiles_rect, two ? L.rowsq : (double*)nullptr);
    hipLaunchKernelGGL(lazy_fix_z_kernel, dim3(mb, LAZY_TM / FIX_SPB), dim3(256), 0, s, L, t.Z, d.m, t.ctrl);
  };
  if (two) update_z();
  {                                     // E = C0 M^-1 (entered in the log of matrix products like the general kernel's launches)
    const size_t shmem = (size_t)(LAZY_TM + TE_ROWS) * TE_LD * sizeof(float);
    if ((err = hipFuncSetAttribute(reinterpret_cast<const void*>(thin_e_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem)) != hipSuccess)
      return err;
    int log_slot = -1;
    gemm_log_open(d.d1, LAZY_TM, LAZY_TM, 0, sn, &log_slot);
    hipLaunchKernelGGL(thin_e_kernel, dim3((d.d1 + TE_ROWS - 1) / TE_ROWS), dim3(512), shmem, sn, L, d.d1, t.ctrl);
    gemm_log_close(log_slot, sn);
  }
  hipLaunchKernelGGL(rk_pack_rows_kernel, dim3((16 * dpad + 255) / 256), dim3(256), 0, sn, L.E, d.d1, dpad, Epk);
  if (two && (err = hipStreamWaitEvent(sn, side->fork, 0)) != hipSuccess) return err;
  // N0 -= E C0^T on the lower block triangle (pivot rows and columns are rewritten below)
  hipLaunchKernelGGL(rk_update_kernel, dim3((unsigned)L.n_tiles_sym), dim3(256), 0, sn, Epk, dpad, Cpk, dpad, t.N, (int64_t)d.d1, d.d1, d.d1,
                     L.tiles_sym, (double*)nullptr);
  hipLaunchKernelGGL(lazy_fix_kernel, dim3(rb, LAZY_TM / FIX_SPB), dim3(256), 0, sn, L, t.N, d.d1, t.ctrl);
  if (!two) update_z();
  if (!two) {
    hipLaunchKernelGGL(lazy_reset_kernel, dim3(1), dim3(256), 0, s, L, t.ctrl);
    if ((err = launch_refresh_scores(d, t, s)) != hipSuccess) return err;
    if ((err = launch_candidate_pick(d, t, L, s, mode)) != hipSuccess) return err;
    if ((err = launch_candidate_products(d, t, L, s, mode)) != hipSuccess) return err;
    return launch_picks(d, t, L, s, mode, false);
  }
  // The second stream goes on, once both matrices are final, with the first half of the score refresh (row norms from the
  // stretch sums, diagonal of N0); this one with the products of the picked rows with the new Z0.
  if ((err = hipStreamWaitEvent(s, side->join, 0)) != hipSuccess) return err;      // the pick
  if ((err = here_to_there()) != hipSuccess) return err;
  hipLaunchKernelGGL(norms_from_stretches_kernel, dim3((d.d1 + 255) / 256 + LAZY_TM), dim3(256), 0, sn, L, d.d1, d.m, 2 * ((d.m + 127) / 128),
                     (d.d1 + 255) / 256, t.N, t.Z, t.gram, t.dblk, t.ctrl);
  if ((err = hipEventRecord(side->join, sn)) != hipSuccess) return err;
  if ((err = launch_candidate_products(d, t, L, s, mode)) != hipSuccess) return err;
  if ((err = hipStreamWaitEvent(s, side->join, 0)) != hipSuccess) return err;
  return launch_picks(d, t, L, s, mode, true);
}

// ------------------------------------------------------------------------------------------------
// Block removal: the t <= LAZY_BT rows that one iteration of the nested schedule prunes (Algorithm 1 with p-hat = t-hat:
// all of them scored at the state the iteration starts from) leave as ONE block pivot instead of t pivots in a row.
// With G the picks, b = N0[T, G], X = M^-1 b (tau x t), the current block N_GG = N0[G, G] - b^T X and D = N_GG^-1:
//   Y = D Z_G (t x m), Z_G = Z0[G, :] - X^T Z0[T, :] the current rows;       obj rises by -sum_a <Z_G[a], Y[a]>
//   every other row i: c_i = N[i, G] = N0[i, G] - C0[i, :] X,  Z_i -= c_i Y,  N_ii -= c_i D c_i^T
//   |Z_i|^2 changes by -2 c_i (Y Z_i^T) + c_i (Y Y^T) c_i^T,  Y Z_i^T = W_i - (ZT Y^T)^T C0[i, :]^T,
//   W_i = Z0_i Y^T = D (GbT[G, i] - X^T GbT[T, i])  from the products computed ahead
//   M^-1 grows by the block [[X D X^T, -X D], [-D X^T, D]].
// As for the swaps (swap.hip), nothing of width m is touched: with K the Gram matrix of the base rows and Q = K_TG - K_TT X,
//   Z_G Z_G^T = K_GG - X^T (K_TG + Q),   Y Y^T = D Z_G Z_G^T D,   ZT Y^T = M^-1 Q D.
// Two launches per iteration of t removals: the pick and the algebra by one workgroup, then the rows.  With ZT and Y formed over all
// columns and the pick a launch of its own it was five, 58 us at 8192 x 2048 (t = 10) with what lies between them; now 35.
// ------------------------------------------------------------------------------------------------
constexpr int BT = LAZY_BT;

typedef double lzd4 __attribute__((ext_vector_type(4)));
static_assert(BT == 16, "one 16 x 16 tile of picks");
constexpr int BX_LD = 20;      // doubles per row of the tables of a block's columns: the k of an operand read lie in different banks
constexpr int KLD = LAZY_NC + LAZY_NS;      // row length of K
// Removal lists: of every 64 rows the LIST_N kept ones of smallest removal cost (finite ones only), ascending, lowest index first on
// ties; an entry's number is row * 512 + slot of its products + 1, -1: no entry
constexpr int LIST_ROWS = 64, LIST_N = BT + 1;
static_assert(LAZY_NC + LAZY_NS < 512 && 65536 <= (1 << 22), "row and slot in one int");
// By a workgroup of four waves: sc (INFINITY where the row is not kept) of 64 rows in shared memory, slot of lane's row in the first
// wave; a wave counts the 16 rows of its own that come before the lane's, the first one adds up.  s_cnt: shared memory
__device__ __forceinline__ void write_list(double* __restrict__ val, int32_t* __restrict__ rows, const double* sc, int (*s_cnt)[LIST_ROWS], int row0,
                                           int slot, int lane, int wave) {
  const double x = sc[lane];
  int below = 0;
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int e = wave * 16 + k;
    const double y = sc[e];
    below += (int)((y < x) | ((y == x) & (e < lane)));
  }
  s_cnt[wave][lane] = below;
  __syncthreads();
  if (wave != 0) return;
  below = (s_cnt[0][lane] + s_cnt[1][lane]) + (s_cnt[2][lane] + s_cnt[3][lane]);
  const bool mine = x < INFINITY;
  const int n = (int)__popcll(__ballot(mine));
  if (mine && below < LIST_N) { val[below] = x; rows[below] = (row0 + lane) * 512 + slot + 1; }
  if (lane < LIST_N && lane >= n) { val[lane] = INFINITY; rows[lane] = -1; }
}
// a score as the lists count it: only finite costs of kept rows
__device__ __forceinline__ double list_score(bool kept, double score) { return kept && score < INFINITY ? score : INFINITY; }
__global__ __launch_bounds__(256) void removal_lists_kernel(LazyPtrs L, int d1, const int32_t* __restrict__ kept, double* __restrict__ score,
                                                             const double* __restrict__ gram, const double* __restrict__ dblk, SearchCtrl* ctrl, int refresh) {
  __shared__ double sc[LIST_ROWS];
  __shared__ int s_cnt[4][LIST_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, row = blockIdx.x * LIST_ROWS + lane, rc = min(row, d1 - 1);
  const int slot = L.cslot[rc];
  if (tid < LIST_ROWS) sc[tid] = row < d1 ? list_score(kept[rc] != 0, refresh ? fresh_score(rc, kept, gram, dblk, score, ctrl) : score[rc]) : INFINITY;
  if (refresh && blockIdx.x == 0) empty_pending(L, ctrl, 256);
  __syncthreads();
  write_list(L.lval + (int64_t)blockIdx.x * LIST_N, L.lrow + (int64_t)blockIdx.x * LIST_N, sc, s_cnt, blockIdx.x * LIST_ROWS, slot, lane, tid >> 6);
}
int removal_list_count(int64_t d1) { return (int)((d1 + LIST_ROWS - 1) / LIST_ROWS); }
hipError_t launch_removal_lists(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, bool refresh) {
  hipLaunchKernelGGL(removal_lists_kernel, dim3(removal_list_count(d.d1)), dim3(256), 0, s, L, d.d1, t.kept, t.score, t.gram, t.dblk, t.ctrl,
                     refresh ? 1 : 0);
  return hipGetLastError();
}

// One workgroup: the t cheapest removals from the lists (own_pick; else the picks are in `pick`), then B = N0[T, G], X = M^-1 B,
// Q = K_TG - K_TT X, P = M^-1 Q, D = (N0[G, G] - B^T X)^-1 (negative definite: minus a principal block of a positive definite inverse),
// Y Y^T and U = P D.  Bound by round trips to memory (lists, picks' rows), by what one compute unit can fetch of M^-1 and K_TT (requested
// first, and only the 32-row blocks that can be pending: all 256 KB took 8 us), the counting of the pick and the inversion of 16 x 16
// (by the last wave, beside the others' product with M^-1; its own rows, the last sixteen pending pivots, come after it).  A wave has
// 16 rows of M^-1 and of K_TT in registers as matrix-core operands.
constexpr int PREP_T = 512, PREP_LISTS = 1024;
__global__ __launch_bounds__(PREP_T) void blk_prep_kernel(LazyPtrs L, const float* __restrict__ N0, int d1, int t, int own_pick, int nlists, int tau_most,
                                                           int32_t* __restrict__ pick, float* __restrict__ gap, const int32_t* __restrict__ kept,
                                                           SearchCtrl* ctrl, int32_t* __restrict__ trace_out) {
  // the tables of the algebra, and before it the lists
  constexpr int HEADS = 128, CAND = LIST_N * LIST_N * (PREP_LISTS / HEADS);
  constexpr int TAB = LAZY_TM * BX_LD, SUM = 8 * BT * (BT + 1), POOL = 3 * TAB + 2 * SUM, LDS_ENT = POOL * 2 / 3 / 8 * 8;
  __shared__ __attribute__((aligned(16))) double pool[POOL];
  double *sb = pool, *sx = pool + TAB, *sq = pool + 2 * TAB;
  double (*sS)[BT][BT + 1] = reinterpret_cast<double (*)[BT][BT + 1]>(pool + 3 * TAB);
  double (*sZ)[BT][BT + 1] = sS + 8;
  double* lv = pool;
  int* ln = reinterpret_cast<int*>(pool + LDS_ENT);
  __shared__ double sD[BT][BT + 1], sW[BT][BT + 1], s_h[HEADS], s_cv[CAND];
  __shared__ int s_pick[BT], sts[LAZY_TM], s_hi[HEADS], s_ci[CAND], s_n, s_bi;
  __shared__ double s_bv, s_edge[2];
  if (ctrl->done | ctrl->pause) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const int tau = tau_all(ctrl);      // every thread reads before thread 0 folds the increment in (after a barrier)
  const int E = min(LIST_N, LDS_ENT / nlists);      // entries of each list that fit (all up to 30000 rows); the others are read where they lie
  if (own_pick) {
    for (int i0 = tid; i0 < nlists * E; i0 += 5 * PREP_T) {
      double x[5];
      int n[5];
#pragma unroll
      for (int u = 0; u < 5; u++) {
        const int i = min(i0 + u * PREP_T, nlists * E - 1);
        const int64_t at = E == LIST_N ? i : (int64_t)(i / E) * LIST_N + i % E;
        x[u] = L.lval[at]; n[u] = L.lrow[at];
      }
#pragma unroll
      for (int u = 0; u < 5; u++) if (i0 + u * PREP_T < nlists * E) { lv[i0 + u * PREP_T] = x[u]; ln[i0 + u * PREP_T] = n[u]; }
    }
  }
  if (tid < LAZY_TM) sts[tid] = tid < tau ? L.tslot[tid] : 0;
  double2 mv[16], kv[16];                                 // row 16 wave + lc of M^-1 and K_TT, columns 8 u + 2 lr, + 1
  const int mrow = wave * 16 + lc;
  const int th = min(LAZY_TM, (tau_most + 31) & ~31);
#pragma unroll
  for (int u0 = 0; u0 < 16; u0 += 4)
    if (wave * 16 < th && 8 * u0 < th)
#pragma unroll
      for (int u = u0; u < u0 + 4; u++) mv[u] = *reinterpret_cast<const double2*>(L.Minv + mrow * LAZY_TM + 8 * u + 2 * lr);
#pragma unroll
  for (int u0 = 0; u0 < 16; u0 += 4)
    if (wave * 16 < th && 8 * u0 < th)
#pragma unroll
      for (int u = u0; u < u0 + 4; u++) kv[u] = *reinterpret_cast<const double2*>(L.KT + mrow * LAZY_TM + 8 * u + 2 * lr);
  if (own_pick) {
    // (value, number) pairs are ordered by value, then number (the lowest row first).  The bound: of the least entries of HEADS groups of
    // lists the (t + 1)-th, found by counting; no entry above it is among the t + 1 smallest.  Then the entries up to it, ranked by counting.
    auto before = [](double x, int i, double y, int j) { return (x < y) | ((x == y) & (i < j)); };
    __syncthreads();
    if (tid < HEADS) {
      double hv = INFINITY;
      int hn = 0x7fffffff - HEADS + tid;                  // no entry: behind all others, each another number
      for (int l = tid; l < nlists; l += HEADS) if (ln[l * E] >= 0 && before(lv[l * E], ln[l * E], hv, hn)) { hv = lv[l * E]; hn = ln[l * E]; }
      s_h[tid] = hv; s_hi[tid] = hn;
    }
    if (tid == 0) { s_n = 0; s_edge[0] = s_edge[1] = INFINITY; }
    if (tid < BT) s_pick[tid] = -1;
    __syncthreads();
    {
      const int h = tid >> 2;                             // four threads to a head
      const double x = s_h[h];
      const int xi = s_hi[h];
      int below = 0;
#pragma unroll 8
      for (int k = 0; k < HEADS / 4; k++) { const int e = (tid & 3) * (HEADS / 4) + k; below += (int)before(s_h[e], s_hi[e], x, xi); }
      below += __builtin_amdgcn_update_dpp(0, below, 0xb1, 0xf, 0xf, true);
      below += __builtin_amdgcn_update_dpp(0, below, 0x4e, 0xf, 0xf, true);
      if ((tid & 3) == 0 && below == t) { s_bv = x; s_bi = xi; }      // t < HEADS: one of them
    }
    __syncthreads();
    const double bound = s_bv;
    const int bound_i = s_bi;
    for (int l = tid; l < nlists; l += PREP_T)
      for (int e = 0; e < LIST_N; e++) {
        const double x = e < E ? lv[l * E + e] : L.lval[(int64_t)l * LIST_N + e];
        const int n = e < E ? ln[l * E + e] : L.lrow[(int64_t)l * LIST_N + e];
        if (n < 0 || before(bound, bound_i, x, n)) break;
        const int at = atomicAdd(&s_n, 1);
        s_cv[at] = x; s_ci[at] = n;                       // t + 1 <= LIST_N groups have a head up to the bound: CAND is enough
      }
    __syncthreads();
    const int found = s_n;
    for (int i = tid; i < found; i += PREP_T) {
      const double x = s_cv[i];
      const int xi = s_ci[i];
      int rank = 0;
      for (int k = 0; k < found; k++) rank += (int)before(s_cv[k], s_ci[k], x, xi);
      if (rank < t) s_pick[rank] = xi;
      if (rank == t - 1) s_edge[0] = x;
      if (rank == t) s_edge[1] = x;
    }
    __syncthreads();
    if (tid < t) { const int c = s_pick[tid]; pick[tid] = c < 0 ? -1 : c >> 9; }
    if (tid == 0) *gap = found > t ? (float)(fabs(s_edge[1] - s_edge[0]) / fmax(fabs(s_edge[0]), 1e-300)) : INFINITY;
  } else if (tid < t) {
    const int g = pick[tid];
    s_pick[tid] = (g >= 0 && g < d1) ? g * 512 + L.cslot[g] + 1 : -1;
  }
  __syncthreads();
  // every wave holds all the picks; what depends on them in one round trip
  const int n = s_pick[lane < t ? lane : 0], g = n >= 0 ? n >> 9 : 0, slot = n >= 0 ? max((n & 511) - 1, 0) : 0;
  const int gl = __shfl(g, lc < t ? lc : 0, 64), sl = __shfl(slot, lc < t ? lc : 0, 64);      // the pick of column lc
  const int kept_g = kept[g], pos_g = L.pos[g];
  double kq[4], kgg[4], x4[4], p4[4];
  float raw[4], n0[4];
#pragma unroll
  for (int r = 0; r < 4; r++) {      // rows of b and K_TG, the picks' own block of N0 and K
    const int k = wave * 16 + 4 * r + lr, a = 4 * r + lr, ga = __shfl(g, a < t ? a : 0, 64), sa = __shfl(slot, a < t ? a : 0, 64);
    raw[r] = L.C0R[(int64_t)gl * LAZY_TM + k];
    kq[r] = L.K[sts[k] * KLD + sl];
    n0[r] = nsym1(N0, d1, ga, gl); kgg[r] = L.K[sa * KLD + sl];
  }
  const bool bad = n < 0 || (n & 511) == 0 || !kept_g || pos_g >= 0 || tau + t > LAZY_TM;
  if (__any(bad)) {                                       // the same in every wave: none writes before all have read
    __syncthreads();
    if (tid == 0) { ctrl->tau = tau; ctrl->tau_inc = 0; ctrl->pause = 1; }
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int k = wave * 16 + 4 * r + lr;
    const bool use = k < tau && lc < t;
    sb[k * BX_LD + lc] = use ? (double)raw[r] : 0.0;
    if (!use) kq[r] = 0.0;
  }
  __syncthreads();
  if (tid == 0) { ctrl->tau = tau; ctrl->tau_inc = 0; }
  auto product = [&](const double2* A, const double* B) {
    lzd4 x = {0.0, 0.0, 0.0, 0.0};
    if (wave * 16 >= tau) return x;
#pragma unroll
    for (int u = 0; u < 16; u++) {                        // B is zero from tau on, the matrices are finite there
      if (8 * u >= tau) break;
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(A[u].x, B[(8 * u + 2 * lr) * BX_LD + lc], x, 0, 0, 0);
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(A[u].y, B[(8 * u + 2 * lr + 1) * BX_LD + lc], x, 0, 0, 0);
    }
    return x;
  };
  {
    const lzd4 x = product(mv, sb);
    lzd4 p = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = wave * 16 + 4 * r + lr;
      x4[r] = row < tau ? x[r] : 0.0;
      sx[row * BX_LD + lc] = x4[r]; L.bX[row * BT + lc] = x4[r];
      p = __builtin_amdgcn_mfma_f64_16x16x4f64(sb[row * BX_LD + lc], x4[r], p, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; r++) sS[wave][4 * r + lr][lc] = p[r];
  }
  __syncthreads();
  {
    const lzd4 q = product(kv, sx);
    lzd4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = wave * 16 + 4 * r + lr;
      const double v = row < tau ? kq[r] - q[r] : 0.0;
      sq[row * BX_LD + lc] = v;
      z = __builtin_amdgcn_mfma_f64_16x16x4f64(x4[r], kq[r] + v, z, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; r++) sZ[wave][4 * r + lr][lc] = z[r];
  }
  __syncthreads();
  if (wave == 7) {
    swd4 y;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int a = 4 * r + lr;
      double v = (double)n0[r], z = kgg[r];
#pragma unroll
      for (int w = 0; w < 8; w++) { v -= sS[w][a][lc]; z -= sZ[w][a][lc]; }
      y[r] = (a < t && lc < t) ? -v : (a == lc ? 1.0 : 0.0);
      sW[a][lc] = (a < t && lc < t) ? z : 0.0;            // Z_G Z_G^T
    }
    bool flag = false;
    inv16(y, lane, t, flag);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int a = 4 * r + lr;
      const double v = (a < t && lc < t) ? -y[r] : 0.0;
      sD[a][lc] = v; L.bD[a * BT + lc] = v;
    }
    if (lane < BT) L.bG[lane] = lane < t ? g : -1;
    if (__any(flag) && lane == 0) ctrl->notpd = 1;
  }
  {
    const lzd4 p = product(mv, sq);
#pragma unroll
    for (int r = 0; r < 4; r++) p4[r] = wave * 16 + 4 * r + lr < tau ? p[r] : 0.0;
  }
  __syncthreads();
  // the tables of Q have been read: P takes their place as an operand (rows = picks of D to contract)
  {
#pragma unroll
    for (int r = 0; r < 4; r++) sq[(wave * 16 + 4 * r + lr) * BX_LD + lc] = p4[r];      // this wave's rows only
    asm volatile("" ::: "memory");      // (a wave's shared-memory operations are in order; the compiler must keep them so)
    lzd4 u = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; k++) u = __builtin_amdgcn_mfma_f64_16x16x4f64(sq[(wave * 16 + lc) * BX_LD + 4 * k + lr], sD[4 * k + lr][lc], u, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; r++) L.bU[(wave * 16 + 4 * r + lr) * BT + lc] = u[r];
    // K_TT grows by the picks
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int k = wave * 16 + 4 * r + lr;
      if (k < tau && lc < t) { L.KT[k * LAZY_TM + tau + lc] = kq[r]; L.KT[(tau + lc) * LAZY_TM + k] = kq[r]; }
    }
  }
  if (wave == 7) {
    lzd4 dz = {0.0, 0.0, 0.0, 0.0}, yy = dz;
#pragma unroll
    for (int k = 0; k < 4; k++) dz = __builtin_amdgcn_mfma_f64_16x16x4f64(sD[lc][4 * k + lr], sW[4 * k + lr][lc], dz, 0, 0, 0);      // D Z_G Z_G^T
    double dsum = 0.0;                                    // sum_a <Z_G[a], Y[a]>: its trace
#pragma unroll
    for (int r = 0; r < 4; r++) { if (4 * r + lr == lc) dsum += dz[r]; if (4 * r + lr < t && lc < t) L.KT[(tau + 4 * r + lr) * LAZY_TM + tau + lc] = kgg[r]; }
    dsum = wsum(dsum);
#pragma unroll
    for (int r = 0; r < 4; r++) sW[4 * r + lr][lc] = dz[r];      // (read above by this wave alone)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 4; k++) yy = __builtin_amdgcn_mfma_f64_16x16x4f64(sW[lc][4 * k + lr], sD[4 * k + lr][lc], yy, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; r++) L.bYY[(4 * r + lr) * BT + lc] = yy[r];
    if (lane == 0) {
      const int it = ctrl->iters;
      ctrl->obj = ctrl->obj - dsum;            // D is negative definite: the objective rises
      ctrl->iters = it + t; ctrl->accepted += t; ctrl->tau_inc = t;
      if (trace_out) for (int a = 0; a < t; a++) trace_out[it + a] = s_pick[a] >> 9;
    }
  }
}

// Rows: the sums over the pending pivots, D wt and the two quadratic forms of every row on v_mfma_f64_16x16x4_f64.  A wave takes 16
// rows, lane (lr, lc) holds the picks 4 r + lr of row lc; a workgroup of 64 rows leaves their removal list.  As 8 lanes per
// row, with the forms left to one of them, a removal of 10 of 8192 rows took 35 us here.
__global__ __launch_bounds__(256) void blk_update_kernel(LazyPtrs L, const float* __restrict__ N0, int d1, int t, int row_groups,
                                                          int row_wgs, SearchCtrl* ctrl, int32_t* __restrict__ kept,
                                                          double* __restrict__ rho, double* __restrict__ diag,
                                                          double* __restrict__ score) {
  __shared__ double sX[LAZY_TM * BX_LD], sU[LAZY_TM * BX_LD], sD[BT * BT], sYY[BT * BT];
  __shared__ int sts[LAZY_TM], sG[BT], sSlot[BT];
  __shared__ double s_sc[LIST_ROWS];
  __shared__ int s_cnt[4][LIST_ROWS];
  if ((ctrl->done | ctrl->pause) != 0) return;
  const int tid = threadIdx.x, tau = ctrl->tau, b = blockIdx.x;
  if (b < row_wgs) {
    for (int idx = tid; idx < (tau + 15) / 16 * 16 * BT; idx += 256) {      // what the loop below reads: zero from tau on
      const int r = idx / BT, a = idx % BT;
      sX[r * BX_LD + a] = L.bX[idx]; sU[r * BX_LD + a] = L.bU[idx];
    }
    for (int idx = tid; idx < BT * BT; idx += 256) { const int a = idx / BT, c = idx % BT; sD[idx] = L.bD[idx]; sYY[idx] = (a < t && c < t) ? L.bYY[idx] : 0.0; }
    for (int s = tid; s < LAZY_TM; s += 256) sts[s] = (s < tau) ? L.tslot[s] : 0;
    if (tid < BT) { const int g = tid < t ? L.bG[tid] : 0; sG[tid] = g; sSlot[tid] = (tid < t) ? L.cslot[g] : 0; }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
    // a workgroup walks groups of 64 rows (a removal list each), so the tables above are loaded once for several
    for (int grp = b; grp < row_groups; grp += row_wgs) {
      const int row = grp * 64 + wave * 16 + lc, rc = min(row, d1 - 1);
      // requested first: the base entries N0[row, G] (new columns of C0), the products GbT[G, row], the row's own values
      float n0[4];
      double gb0[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int a = 4 * r + lr;
        n0[r] = nsym1(N0, d1, rc, sG[a]);
        gb0[r] = L.GbT[(int64_t)sSlot[a] * d1 + rc];
      }
      const int ps = L.pos[rc], kp0 = kept[rc], slot0 = L.cslot[min(grp * LIST_ROWS + lane, d1 - 1)];
      const double rho0 = rho[rc], diag0 = diag[rc];
      lzd4 dx = {0.0, 0.0, 0.0, 0.0}, du = dx, dw = dx;
      const float* crow = L.C0R + (int64_t)rc * LAZY_TM;
      for (int k0 = 0; k0 < tau; k0 += 16) {              // k = k0 + 4 lr + e: a lane's four values of C0 are one load
        const float4 c4 = *reinterpret_cast<const float4*>(crow + k0 + 4 * lr);
        const float ce[4] = {c4.x, c4.y, c4.z, c4.w};
        double gv[4];
#pragma unroll
        for (int e = 0; e < 4; e++) gv[e] = L.GbT[(int64_t)sts[k0 + 4 * lr + e] * d1 + rc];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int k = k0 + 4 * lr + e;
          const double x = sX[k * BX_LD + lc], u = sU[k * BX_LD + lc];      // zero from tau on
          const double c = k < tau ? (double)ce[e] : 0.0;
          dx = __builtin_amdgcn_mfma_f64_16x16x4f64(x, c, dx, 0, 0, 0);
          du = __builtin_amdgcn_mfma_f64_16x16x4f64(u, c, du, 0, 0, 0);
          dw = __builtin_amdgcn_mfma_f64_16x16x4f64(x, k < tau ? gv[e] : 0.0, dw, 0, 0, 0);
        }
      }
      lzd4 w = {0.0, 0.0, 0.0, 0.0}, sy = w, sd = w;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int a = 4 * r + lr;
        w = __builtin_amdgcn_mfma_f64_16x16x4f64(sD[lc * BT + a], a < t ? gb0[r] - dw[r] : 0.0, w, 0, 0, 0);
        if (a < t && row < d1) L.C0R[(int64_t)row * LAZY_TM + tau + a] = n0[r];
      }
      double cg[4], zy[4];
      const double sg = ps >= 0 ? (double)L.Jsg[ps] : 0.0;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int a = 4 * r + lr;
        cg[r] = a >= t ? 0.0 : ps >= 0 ? sg * sX[ps * BX_LD + a] : (double)n0[r] - dx[r];
        zy[r] = a >= t ? 0.0 : ps >= 0 ? sg * sU[ps * BX_LD + a] : w[r] - du[r];
      }
#pragma unroll
      for (int r = 0; r < 4; r++) {
        sy = __builtin_amdgcn_mfma_f64_16x16x4f64(sYY[lc * BT + 4 * r + lr], cg[r], sy, 0, 0, 0);
        sd = __builtin_amdgcn_mfma_f64_16x16x4f64(sD[lc * BT + 4 * r + lr], cg[r], sd, 0, 0, 0);
      }
      double lin = 0, quadY = 0, quadD = 0;
#pragma unroll
      for (int r = 0; r < 4; r++) { lin += cg[r] * zy[r]; quadY += cg[r] * sy[r]; quadD += cg[r] * sd[r]; }
      lin += __shfl_xor(lin, 16, 64); quadY += __shfl_xor(quadY, 16, 64); quadD += __shfl_xor(quadD, 16, 64);
      lin += __shfl_xor(lin, 32, 64); quadY += __shfl_xor(quadY, 32, 64); quadD += __shfl_xor(quadD, 32, 64);
      if (lr == 0) {
        int kp = -1;
        double sc = 0.0;
        if (row < d1) {
          int mine = -1;
          for (int a = 0; a < t; a++) if (sG[a] == row) mine = a;
          double r, dn;
          if (mine >= 0) {
            r = sYY[mine * BT + mine]; dn = -sD[mine * BT + mine]; kp = 0;
            L.pos[row] = tau + mine; L.Tidx[tau + mine] = row; L.Jsg[tau + mine] = -1.f; L.tslot[tau + mine] = sSlot[mine];
          } else {
            r = rho0 - 2.0 * lin + quadY;
            if (r < 0.0) r = 0.0;
            dn = diag0 - quadD;
            kp = kp0;
          }
          rho[row] = r; diag[row] = dn; kept[row] = kp;
          sc = r / fabs(dn);
          score[row] = sc;
        }
        s_sc[wave * 16 + lc] = list_score(kp > 0, sc);
      }
      __syncthreads();
      write_list(L.lval + (int64_t)grp * LIST_N, L.lrow + (int64_t)grp * LIST_N, s_sc, s_cnt, grp * LIST_ROWS, slot0, lane, wave);
      __syncthreads();
    }
  } else {
    const int mb = b - row_wgs, nmb = gridDim.x - row_wgs;
    double* Mi = L.Minv;
    // M^-1 += X D X^T: a wave per lower 16 x 16 tile (mirrored, so that M^-1 stays symmetric to the bit)
    const int lane = tid & 63, lr = lane >> 4, lc = lane & 15;
    for (int tile = mb * 4 + (tid >> 6); tile < 36; tile += nmb * 4) {
      int I = 0, J = tile;
      while (J > I) { J -= I + 1; I++; }
      if (I * 16 >= tau) break;
      lzd4 dx = {0.0, 0.0, 0.0, 0.0}, v = dx;
#pragma unroll
      for (int r = 0; r < 4; r++) dx = __builtin_amdgcn_mfma_f64_16x16x4f64(L.bD[lc * BT + 4 * r + lr], L.bX[(J * 16 + lc) * BT + 4 * r + lr], dx, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; r++) v = __builtin_amdgcn_mfma_f64_16x16x4f64(L.bX[(I * 16 + lc) * BT + 4 * r + lr], dx[r], v, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int i = I * 16 + 4 * r + lr, j = J * 16 + lc;
        if (i >= tau || j > i) continue;
        const double m2 = Mi[i * LAZY_TM + j] + v[r];
        Mi[i * LAZY_TM + j] = m2; Mi[j * LAZY_TM + i] = m2;
      }
    }
    if (mb == 0) {
      for (int idx = tid; idx < tau * t; idx += 256) {
        const int r = idx / t, a = idx % t;
        double v = 0;
        for (int bb = 0; bb < t; bb++) v -= L.bX[r * BT + bb] * L.bD[bb * BT + a];
        Mi[r * LAZY_TM + tau + a] = v; Mi[(tau + a) * LAZY_TM + r] = v;
      }
      for (int idx = tid; idx < t * t; idx += 256) { const int a = idx / t, bb = idx % t; Mi[(tau + a) * LAZY_TM + tau + bb] = L.bD[a * BT + bb]; }
    }
  }
}

hipError_t launch_lazy_block_remove(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, int take, bool own_pick, int tau_most, int32_t* pick,
                                    float* gap, hipStream_t s) {
  if (take < 1 || take > BT || removal_list_count(d.d1) > PREP_LISTS) return hipErrorInvalidValue;
  hipLaunchKernelGGL(blk_prep_kernel, dim3(1), dim3(PREP_T), 0, s, L, t.N, d.d1, take, own_pick ? 1 : 0, removal_list_count(d.d1), tau_most, pick, gap, t.kept,
                     t.ctrl, t.trace_out);
  const int rg = (d.d1 + 63) / 64, row_wgs = std::min(rg, 256);
  hipLaunchKernelGGL(blk_update_kernel, dim3(row_wgs + 16), dim3(256), 0, s, L, t.N, d.d1, take, rg, row_wgs, t.ctrl, t.kept, t.gram, t.dblk, t.score);
  return hipGetLastError();
}

hipError_t launch_lazy_init(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode) {
  hipError_t e = hipMemsetAsync(L.pos, 0xFF, (size_t)d.d1 * 4, s);
  if (e != hipSuccess) return e;
  for (double* M : {L.Minv, L.Minv2, L.KT})      // finite beyond the pending pivots
    if ((e = hipMemsetAsync(M, 0, (size_t)LAZY_TM * LAZY_TM * 8, s)) != hipSuccess) return e;
  e = hipMemsetAsync(L.C0R, 0, (size_t)d.d1 * LAZY_TM * 4, s);
  if (e != hipSuccess) return e;
  if ((e = launch_candidate_pick(d, t, L, s, mode)) != hipSuccess || (e = launch_candidate_products(d, t, L, s, mode)) != hipSuccess) return e;
  return launch_picks(d, t, L, s, mode, false);
}

}  // namespace osscar
