// One swap of the delayed-update search (q = 1) in one launch: swaps that fetch products, removals, and layers or GPUs on which the workgroups
// of many swaps in one launch (swaprun.hip) are not resident together.
//
// The tableau in HBM stays at its base state (N0, Z0) between two flushes; T is the set of pivots swept since, M = N0[T, T], x_h = M^-1
// N0[T, h] (lazy.hip has the algebra).  The current row h of Z is z_h = Z0[h] - x_h^T Z0[T], so every inner product that a swap of
// (g, j) needs follows from x_g, x_j and the float64 Gram matrix K of the base rows that can become pivots (the rows whose products
// with all of Z0 are computed ahead, and those fetched since):
//     z_a . z_b = K_ab - x_a . K_Tb - x_b . (K_Ta - K_TT x_a),       ZT z_a = M^-1 (K_Ta - K_TT x_a),       ZT = M^-1 Z0[T].
// Nothing of width m is touched: the change of the objective, the acceptance test, u = ZT [y1 y2] and |y1|^2, y1 . y2, |y2|^2 are
// algebra of order |T| <= 128.  It is small enough for every workgroup to do it for itself (M^-1 and K_TT are requested before the
// pivots are known and wait in registers), so a swap is one launch without a one-workgroup phase in front:
//     pick from the workgroups' records | rows g, j of C0, the products' columns | x | K_T. - K_TT x | ZT z | the workgroup's rows
// What every workgroup reads and one of them writes (control block, M^-1, records) has two copies: every launch reads one and writes
// the other, also where it makes no swap, so that nothing has to be read before the addresses of the first requests are known.  What only grows (C0, K_TT, the pending lists) is read below tau and written from tau on.
// Bound by latency: three dependent round trips to memory (records, pivots' rows, launch to launch), five barriers and three products
// of a 128 x 128 matrix with two vectors; at 28672 rows also by what the rows read (15 MB of products and 7 MB of C0 on average).  As four
// launches, the first of them one workgroup, with ZT (128 x m) updated and read by every swap, a swap took 25 us at 8192 x 2048 (flushes
// and waits apart) and 31 at 28672 x 7168; in one launch 11 and 21.
#include "internal.h"
#include "lazy_device.h"
#include "wave.h"
#include <algorithm>

namespace osscar {

constexpr int KLD = LAZY_NC + LAZY_NS;      // row length of K
constexpr int PENDING = 1 << 30;            // flag in a record's slot: the row is a pending pivot
constexpr int LIST_MOST = 64;               // pairs (rows) of a list: one per lane

// p[i] with a byte offset of 32 bits (C0: 65536 rows of 512 bytes; the products: 320 rows of 65536 doubles)
template <typename T>
__device__ __forceinline__ T at32(const T* p, uint32_t i) { return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + i * (uint32_t)sizeof(T)); }

// Best and second best of a block of RPW rows, cheapest removal by wave 0, largest gain by wave 1; sc, kp (1 kept, 0 not, -1 no row)
// and sl (slot, or PENDING) in shared memory.  A row whose score is NaN is none of them (which of the others were compared with it, and lost,
// would depend on the lanes).
template <int RPW>
__device__ __forceinline__ void write_record(SwapRec* rec, const double* sc, const int* kp, const int* sl, int row0, int wave, int lane) {
  constexpr int E = (RPW + 63) / 64;
  if (wave > 1) return;
  double own[E], v = INFINITY;
  int idx[E], i = -1;
#pragma unroll
  for (int e = 0; e < E; e++) {
    const int k = lane + 64 * e;
    const double s = sc[k < RPW ? k : 0];
    const bool has = k < RPW && kp[k < RPW ? k : 0] == 1 - wave && s == s;
    own[e] = has ? (wave == 0 ? s : -s) : INFINITY;
    idx[e] = has ? row0 + k : -1;
    if (idx[e] >= 0 && (i < 0 || own[e] < v)) { v = own[e]; i = idx[e]; }
  }
  wave_min(v, i);
  const int win = __builtin_amdgcn_readlane(i, 63);
  double second = INFINITY;
#pragma unroll
  for (int e = 0; e < E; e++) if (idx[e] >= 0 && idx[e] != win) second = fmin(second, own[e]);
  second = wave_min(second);
  if (lane == 63) {
    rec->best[wave] = v; rec->second[wave] = second;
    rec->row[wave] = win; rec->slot[wave] = win >= 0 ? sl[win - row0] : -1;
  }
}

// the records of the scores as they stand (nothing pending); refresh: of the scores from the norms and the diagonal, after a flush.
// Clears the `words` shared words of the runs of swaps.
template <int RPW>
__global__ __launch_bounds__(128) void swap_records_kernel(LazyPtrs L, int d1, const int32_t* __restrict__ kept, double* __restrict__ score,
                                                            const double* __restrict__ gram, const double* __restrict__ dblk, SearchCtrl* ctrl, int refresh, uint64_t* __restrict__ shared, int words) {
  __shared__ double sc[RPW];
  __shared__ int kp[RPW], sl[RPW];
  const int tid = threadIdx.x, row = blockIdx.x * RPW + tid;
  for (int i = blockIdx.x * 128 + tid; i < words; i += gridDim.x * 128) shared[i] = 0;
  if (tid < RPW) {
    const bool in = row < d1;
    sc[tid] = !in ? 0.0 : refresh ? fresh_score(row, kept, gram, dblk, score, ctrl) : score[row]; kp[tid] = in ? (kept[row] != 0) : -1; sl[tid] = in ? L.cslot[row] : -1;
  }
  __syncthreads();
  if (refresh && blockIdx.x == 0) empty_pending(L, ctrl, 128);
  write_record<RPW>(L.rec + blockIdx.x, sc, kp, sl, blockIdx.x * RPW, tid >> 6, tid & 63);
}

// A pivot whose products were not computed ahead: its column of Z0 Z0^T by a pass over the workgroup's rows, its row of K by dot products
// with the rows in the other slots, a wave each (products and sums in float64).  miss: 1 for g, 2 for j, slots sg, sj; `used` slots of K
// beyond the picked rows are taken once these are in.  Bound by memory where the rows fill the chip; with few of them, by the chain of
// requests that a wave makes along a row, so rows of any length are read four columns a lane.  Column by column where the length is no
// multiple of four, and with one request of a row of K in flight, all of them by neighbouring workgroups: 28672 x 7168, every pivot
// fetched, 318 us a swap, 228 so; 1000 x 4093 79 us, 41 so (a fetch and a swap each, and the flushes).
typedef float row4 __attribute__((ext_vector_type(4), aligned(4)));      // four columns of a row of any length
template <int NT>
__device__ __forceinline__ void fetch_products(const LazyPtrs& L, const float* __restrict__ Z0, int d1, int m, int g, int j, int miss, int sg, int sj,
                                               int used) {
  constexpr int W = NT / 64, R = 4, UN = NT == 512 ? 4 : 1;      // (more, or in arrays: the kernel spills, and the swaps that fetch nothing are slower)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wg = blockIdx.x, nwg = gridDim.x;
  const float *yg = Z0 + (int64_t)g * m, *yj = Z0 + (int64_t)j * m;
  const int m4 = m & ~3;
  const int per = (d1 + R * nwg - 1) / (R * nwg) * R;      // neighbouring rows, as the lines that they are written to
  for (int r0 = wg * per + wave * R; r0 < min(d1, (wg + 1) * per); r0 += W * R) {
    double a[R], b[R];
    const float* rp[R];
#pragma unroll
    for (int r = 0; r < R; r++) { a[r] = 0; b[r] = 0; rp[r] = Z0 + (int64_t)min(r0 + r, d1 - 1) * m; }
#pragma unroll UN
    for (int c = lane * 4; c < m4; c += 256) {
      const row4 p = *reinterpret_cast<const row4*>(yg + c), q = *reinterpret_cast<const row4*>(yj + c);
#pragma unroll
      for (int r = 0; r < R; r++) {
        const row4 v = *reinterpret_cast<const row4*>(rp[r] + c);
#pragma unroll
        for (int e = 0; e < 4; e++) { a[r] += (double)v[e] * (double)p[e]; b[r] += (double)v[e] * (double)q[e]; }
      }
    }
    if (m4 + lane < m) {
      const double p = yg[m4 + lane], q = yj[m4 + lane];
#pragma unroll
      for (int r = 0; r < R; r++) { const double v = rp[r][m4 + lane]; a[r] += v * p; b[r] += v * q; }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
      const double t = wsum(a[r]), u = wsum(b[r]);
      const int row = r0 + r;
      if (lane == 0 && row < d1) {
        if (miss & 1) L.GbT[(int64_t)sg * d1 + row] = t;
        if (miss & 2) L.GbT[(int64_t)sj * d1 + row] = u;
      }
    }
  }
  for (int t = wg + nwg * (W - 1 - wave); t < LAZY_NC + used; t += nwg * W) {
    const int h = ((miss & 1) && t == sg) ? g : ((miss & 2) && t == sj) ? j : L.cand[t];
    if (h < 0) continue;
    const float* z = Z0 + (int64_t)h * m;
    double a = 0, b = 0;
    for (int c0 = lane * 4; c0 < m4; c0 += 1024) {      // four requests of each row in flight: a chain of one wave's loads
      row4 v[4], p[4], q[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int c = c0 + 256 * u < m4 ? c0 + 256 * u : 0;
        v[u] = *reinterpret_cast<const row4*>(z + c); p[u] = *reinterpret_cast<const row4*>(yg + c); q[u] = *reinterpret_cast<const row4*>(yj + c);
      }
#pragma unroll
      for (int u = 0; u < 4; u++) {
        if (c0 + 256 * u >= m4) break;
#pragma unroll
        for (int e = 0; e < 4; e++) { a += (double)v[u][e] * (double)p[u][e]; b += (double)v[u][e] * (double)q[u][e]; }
      }
    }
    if (m4 + lane < m) { const double v = z[m4 + lane]; a += v * (double)yg[m4 + lane]; b += v * (double)yj[m4 + lane]; }
    a = wsum(a); b = wsum(b);
    if (lane == 0) {
      if (miss & 1) { L.K[sg * KLD + t] = a; L.K[t * KLD + sg] = a; }
      if (miss & 2) { L.K[sj * KLD + t] = b; L.K[t * KLD + sj] = b; }
    }
  }
}

// NT threads, RPW rows per workgroup, NT / RPW lanes per row.  cin: control block before this launch, cout: after it.
// limit: iterations to have run after this launch at most; beyond it a launch does nothing.  list_n > 0: the last list_n of them take the
// pairs (list_g[r * list_step], list_j[r * list_step]), r = 0, 1, ... (the pick, where an entry of list_g is no row), list_j == nullptr:
// remove the rows of list_g (Case 1 alone).  The launch finds its place in the list by the iterations that have run, so a pair whose
// launch had to fetch products is the next launch's: with a place fixed when it is enqueued, the launches behind a fetch were idle and
// were enqueued again after a wait (layer of 700 rows in moves of 32 pairs: 15.3 ms, so 6.6).  A pair that is not (kept, not
// kept) has no definite pivots and is refused as such.
template <int NT, int RPW>
__global__ __launch_bounds__(NT) void lazy_swap_kernel(LazyPtrs L, const float* __restrict__ N0, const float* __restrict__ Z0, int d1, int m,
                                                        const SearchCtrl* __restrict__ cin, SearchCtrl* __restrict__ cout, int32_t* __restrict__ kept,
                                                        double* __restrict__ rho, double* __restrict__ diag, double* __restrict__ score, int always, int tau_most,
                                                        const int32_t* __restrict__ list_g, const int32_t* __restrict__ list_j, int list_n, int list_step, int limit, int fetch_only, int nwg, int32_t* __restrict__ trace_out,
                                                        int32_t* __restrict__ trace_in, float* __restrict__ trace_gap, double* __restrict__ trace_obj) {
  constexpr int TM = LAZY_TM, W = NT / 64, H = NT / 2;
  constexpr int TPR = NT / TM, MU = TM / (2 * TPR);             // threads per row of M^-1, pairs of columns per thread
  constexpr int UG = 32 / (2 * TPR);                            // 32 columns of it
  constexpr int LPR = NT / RPW, CT = TM / (4 * LPR), GB = TM / LPR;      // lanes per row of the tableau, its loads of C0 and of the products
  static_assert((TPR == 4 || TPR == 8) && (LPR == 8 || LPR == 16) && W >= 8, "reductions below");
  __shared__ double s_v[W], s_2nd[W];
  __shared__ int s_i[W], s_s[W], sts[TM];
  __shared__ __attribute__((aligned(16))) double sb[2][TM], sk[2][TM], sx[2][TM], st[2][TM], sp[2][TM];
  __shared__ double dots[6], s_n0[3], s_kk[3], red[2][LPR][RPW];
  __shared__ double s_sc[RPW];
  __shared__ int s_kp[RPW], s_sl[RPW];
  // 1024 threads have 128 registers each: K_TT waits in shared memory instead, put there by direct loads (rows from tau on: anything)
  constexpr bool KT_LDS = NT == 1024;
  __shared__ __attribute__((aligned(16))) double s_kt[KT_LDS ? TM * TM : 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wg = blockIdx.x;
  const bool helper = wg >= nwg;      // no rows: picks and fetches only
  // ---- requests that do not depend on the pick, in the order in which they are needed (loads return in order); only what can be
  // pending: blocks of 32 rows and columns (the loads of all 128 took 1.8 us at the 64 bytes a cycle that a compute unit receives)
  const int th = helper ? 0 : min(TM, (tau_most + 2 + 31) & ~31);      // this launch's pivots included
  const int side = tid >= H, rt = tid & (H - 1);
  const SwapRec* rp = L.rec + (rt < nwg ? rt : 0);
  double v1 = rp->best[side], v2 = rp->second[side];
  int i1 = rp->row[side], sl1 = rp->slot[side];
  const int ts = tid < TM ? L.tslot[tid] : 0;
  const bool single = list_n > 0 && !list_j;
  const int at = list_n > 0 ? min(lane, list_n - 1) * list_step : 0;      // the whole list (a row each lane): which entry is known later
  const int lg = (list_n > 0 ? list_g : L.cand)[at], lj = (list_n > 0 && list_j ? list_j : L.cand)[at];
  const int mr = tid / TPR, mq = tid % TPR;
  const bool mine = __builtin_amdgcn_readfirstlane(mr) < th;      // 64 / TPR rows a wave: all of them or none
  double2 mv[MU], kv[KT_LDS ? 1 : MU];
#pragma unroll
  for (int u0 = 0; u0 < MU; u0 += UG)
    if (mine && 2 * TPR * u0 < th)
#pragma unroll
      for (int u = u0; u < u0 + UG; u++) mv[u] = *reinterpret_cast<const double2*>(L.Minv + mr * TM + 2 * TPR * u + 2 * mq);
  if constexpr (KT_LDS) {
    for (int r = wave; r < th; r += W)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(L.KT + r * TM + 2 * lane),
                                       (__attribute__((address_space(3))) void*)(s_kt + r * TM), 16, 0, 0);
  } else {
#pragma unroll
    for (int u0 = 0; u0 < MU; u0 += UG)
      if (mine && 2 * TPR * u0 < th)
#pragma unroll
        for (int u = u0; u < u0 + UG; u++) kv[u] = *reinterpret_cast<const double2*>(L.KT + mr * TM + 2 * TPR * u + 2 * mq);
  }
  const int tau = cin->tau, spare = cin->spare;
  // M^-1 is written by all the workgroups: pair u of row mr by workgroup (mr MU + u) mod nwg
  const int own = (wg + nwg - mr * MU % nwg) % nwg;      // the thread's first pair; the next ones nwg further
  auto piece = [&](int u) { return mr * TM + 2 * TPR * u + 2 * mq; };
  auto pass_on = [&](int g, int slot_g, int j, int slot_j) {      // no swap: the state as it stands, with new slots of rows g, j
    for (int u = own; u < MU && mr < th && 2 * TPR * u < th; u += nwg)
      *reinterpret_cast<double2*>(L.Minv2 + piece(u)) = *reinterpret_cast<const double2*>(L.Minv + piece(u));
    if (tid == 0 && !single) {
      SwapRec r = L.rec[wg];
      if (r.row[0] == g) r.slot[0] = slot_g;
      if (r.row[1] == j) r.slot[1] = slot_j;
      L.rec2[wg] = r;
    }
  };
  const bool idle = (cin->done | cin->pause) != 0 || cin->iters >= limit;
  // ---- pick: lanes of the first half of the workgroup hold the leaving side's records, the others the entering side's
  // (the removal-only loops keep lists instead of records: removals of given rows leave the records alone, and their gaps are infinite)
  if (rt >= nwg || single) { v1 = INFINITY; v2 = INFINITY; i1 = -1; sl1 = -1; }
  double wv = v1;
  int wi = i1;
  wave_min(wv, wi);
  wi = __builtin_amdgcn_readlane(wi, 63);
  if (wi >= 0 ? i1 == wi : lane == 0) { s_v[wave] = v1; s_i[wave] = wi; s_s[wave] = sl1; }      // one lane: a row is in one record
  if (tid < TM) sts[tid] = tid < tau ? ts : 0;
  __syncthreads();
  // products of the pending pivots with the rows: row tid % RPW, every LPR-th pivot from tid / RPW on (further down the pivots' own, in
  // slices 0 and 1)
  const int wrow = tid % RPW, wsl = tid / RPW, wrc = min(wg * RPW + wrow, d1 - 1);
  double gb[GB];
  auto request_gb = [&]() {
#pragma unroll
    for (int u0 = 0; u0 < GB; u0 += 32 / LPR)
      if (LPR * u0 < th)
#pragma unroll
        for (int u = u0; u < u0 + 32 / LPR; u++) { const int r = wsl + LPR * u; gb[u] = at32(L.GbT, (uint32_t)sts[r < tau ? r : 0] * d1 + wrc); }
  };
  if (!KT_LDS) { request_gb(); asm volatile("" ::: "memory"); }      // (1024 threads: after the loads that depend on the pick, for the registers)
  // the first W / 2 lanes hold the leaving side's results, the next W / 2 the entering side's
  double qv = s_v[lane & (W - 1)];
  const int qi0 = s_i[lane & (W - 1)], qs0 = s_s[lane & (W - 1)];
  int qi = qi0;
  dpp_min_step<0xb1, 0xf>(qv, qi); dpp_min_step<0x4e, 0xf>(qv, qi);
  if (W == 16) dpp_min_step<0x141, 0xf>(qv, qi);
  int g = __builtin_amdgcn_readlane(qi, 0), j = __builtin_amdgcn_readlane(qi, W / 2);
  const uint64_t has_g = __ballot(lane < W / 2 && qi0 == g), has_j = __ballot(lane >= W / 2 && lane < W && qi0 == j);
  int sg = __builtin_amdgcn_readlane(qs0, has_g ? (int)__builtin_ctzll(has_g) : 0), sj = __builtin_amdgcn_readlane(qs0, has_j ? (int)__builtin_ctzll(has_j) : W / 2);
  const int pick_g = g, pick_j = j;
  const int entry = cin->iters - (limit - list_n), entry_c = __builtin_amdgcn_readfirstlane(min(max(entry, 0), LIST_MOST - 1));
  const int forced_g = (list_n > 0 && entry >= 0) ? __builtin_amdgcn_readlane(lg, entry_c) : -1;
  if (single || forced_g >= 0) {
    g = forced_g; j = single ? g : __builtin_amdgcn_readlane(lj, entry_c);
    if (g < 0 || g >= d1 || j < 0 || j >= d1) { g = -1; j = -1; }
    else {
      // another workgroup may already have entered the row as this launch's pivot (pos = tau) or taken it a slot (from
      // LAZY_NC + spare on): neither counts here
      const int pg = L.pos[g], pj = L.pos[j];
      sg = (pg >= 0 && pg < tau) ? PENDING : L.cslot[g];
      sj = (pj >= 0 && pj < tau) ? PENDING : L.cslot[j];
    }
  }
  g = __builtin_amdgcn_readfirstlane(g); j = __builtin_amdgcn_readfirstlane(j);
  sg = __builtin_amdgcn_readfirstlane(sg); sj = __builtin_amdgcn_readfirstlane(sj);
  const int npiv = single ? 1 : 2;
  const bool hit_g = sg >= 0 && sg < LAZY_NC + spare, hit_j = single ? true : (sj >= 0 && sj < LAZY_NC + spare);
  const bool pending = sg == PENDING || (!single && sj == PENDING);
  const int miss = (hit_g ? 0 : 1) | (hit_j ? 0 : 2), need = (hit_g ? 0 : 1) + (hit_j ? 0 : 1);
  enum { SWAP, IDLE, NONE, PAUSE, FETCH };
  const int act = idle ? IDLE : (g < 0 || j < 0) ? NONE : (pending || tau + npiv > TM || spare + need > LAZY_NS) ? PAUSE : miss ? FETCH : fetch_only ? IDLE : SWAP;
  if (__builtin_expect(act != SWAP, 0)) {      // laid out behind the swap: in between, its code made the swaps 2 % slower
    const int ng = (miss & 1) ? LAZY_NC + spare : sg, nj = (miss & 2) ? LAZY_NC + spare + (miss & 1) : sj;
    if (act == FETCH) fetch_products<NT>(L, Z0, d1, m, g, j, miss, ng, nj, spare + need);      // the next launch finds them
    if (wg == 0 && tid == 0) {
      SearchCtrl c = *cin;
      if (act == NONE) { c.done = 1; c.g_out = -1; c.g_in = -1; }
      if (act == PAUSE) c.pause = 1;
      if (act == FETCH) {
        if (miss & 1) { L.cslot[g] = ng; L.cand[ng] = g; }
        if (miss & 2) { L.cslot[j] = nj; L.cand[nj] = j; }
        c.spare = spare + need; c.misses += need;
      }
      *cout = c;
    }
    if (!helper) pass_on(act == FETCH && (miss & 1) ? g : -2, ng, act == FETCH && (miss & 2) ? j : -2, nj);
    return;
  }
  if (helper) return;
  // ---- everything that depends on the pick, in one round trip (loads without conditions: one under a condition is waited for where
  // the condition ends)
  const int jc = single ? g : j, sjc = single ? sg : sj;
  const int bc = tid & (TM - 1), bh = (tid >> 7) & 1;            // threads 0 - 127: of g, 128 - 255: of j
  const float b_raw = at32(L.C0R, (uint32_t)(bh ? jc : g) * TM + bc);
  const double k_raw = L.K[(bh ? sjc : sg) * KLD + sts[bc]];
  const int e2 = tid & 3, er = e2 == 0 ? g : jc, ec = e2 == 2 ? jc : g;      // threads 256 - 258: (g, g), (j, g), (j, j)
  const float n0_raw = N0[(int64_t)max(er, ec) * d1 + min(er, ec)];
  const double kk_raw = L.K[(e2 == 0 ? sg : sjc) * KLD + (e2 == 2 ? sjc : sg)];
  // the tableau rows, LPR lanes each: the base columns g, j
  const int lr = tid % LPR, row = wg * RPW + tid / LPR, rc = min(row, d1 - 1);
  const float n0g = nsym1(N0, d1, rc, g), n0j = nsym1(N0, d1, rc, jc);
  const double bgj = at32(L.GbT, (uint32_t)(wsl == 1 ? sjc : sg) * d1 + wrc);
  if (KT_LDS) request_gb();
  if (tid < 2 * TM) {
    const bool use = bc < tau && !(bh && single);
    sb[bh][bc] = use ? (double)b_raw : 0.0; sk[bh][bc] = use ? k_raw : 0.0;
  }
  if (tid >= 256 && tid < 259) { s_n0[tid - 256] = (double)n0_raw; s_kk[tid - 256] = kk_raw; }
  if (wg == 0) {      // second-best values: every record's best unless it is the pick
    const double sec = wave_min(i1 >= 0 && i1 != (side ? pick_j : pick_g) ? v1 : v2);
    if (lane == 63) s_2nd[wave] = sec;
  }
  __syncthreads();
  auto matvec = [&](auto A, const double (*x)[TM], double& a, double& b) {
    a = 0; b = 0;
    if (!mine) return;
#pragma unroll
    for (int u = 0; u < MU; u++) {
      if (u % UG == 0 && 2 * TPR * u >= th) break;
      const double2 e = A(u);
      const double2 p = *reinterpret_cast<const double2*>(&x[0][2 * TPR * u + 2 * mq]), q = *reinterpret_cast<const double2*>(&x[1][2 * TPR * u + 2 * mq]);
      a += e.x * p.x + e.y * p.y; b += e.x * q.x + e.y * q.y;
    }
    a += dpp_get<0xb1, 0xf>(a); b += dpp_get<0xb1, 0xf>(b);
    a += dpp_get<0x4e, 0xf>(a); b += dpp_get<0x4e, 0xf>(b);
    if (TPR == 8) { a += dpp_get<0x141, 0xf>(a); b += dpp_get<0x141, 0xf>(b); }
  };
  auto m_of = [&](int u) { return mv[u]; };
  auto k_of = [&](int u) {
    if constexpr (KT_LDS) return *reinterpret_cast<const double2*>(s_kt + mr * TM + 2 * TPR * u + 2 * mq); else return kv[u];
  };
  double ma, mb;
  // x = M^-1 b (b is zero from tau on, M^-1 finite there)
  matvec(m_of, sb, ma, mb);
  if (mq == 0) { sx[0][mr] = mr < tau ? ma : 0.0; sx[1][mr] = mr < tau ? mb : 0.0; }
  if constexpr (KT_LDS) __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));      // vmcnt = 0: K_TT is in shared memory
  __syncthreads();
  // the rows themselves: they arrive while the next products run (columns from tau on: the row's first ones again, not used)
  const double2 mo = *reinterpret_cast<const double2*>(L.Minv + piece(min(own, MU - 1)));
  const int ps = L.pos[rc], kp0 = kept[rc], slot0 = L.cslot[rc];
  const double rho0 = rho[rc], diag0 = diag[rc];
  float4 c4[CT];
#pragma unroll
  for (int t = 0; t < CT; t++) c4[t] = at32(reinterpret_cast<const float4*>(L.C0R), (uint32_t)rc * (TM / 4) + lr + (4 * LPR * t < th ? LPR * t : 0));
  // t = K_T. - K_TT x
  matvec(k_of, sx, ma, mb);
  if (mq == 0) { st[0][mr] = mr < tau ? sk[0][mr] - ma : 0.0; st[1][mr] = mr < tau ? sk[1][mr] - mb : 0.0; }
  // b . x, a wave each
  if (wave >= W - 3) {
    const int k = wave - (W - 3), ib = k >= 1, ix = k == 2;
    const double v = wsum(sb[ib][lane] * sx[ix][lane] + sb[ib][lane + 64] * sx[ix][lane + 64]);
    if (lane == 0) dots[k] = v;
  }
  // the rows' sums over the pending pivots
  {
    double ag = 0, aj = 0;
#pragma unroll
    for (int u = 0; u < GB; u++) { const int r = wsl + LPR * u; if (u % (32 / LPR) == 0 && LPR * u >= th) break; const double v = r < tau ? gb[u] : 0.0; ag += sx[0][r] * v; aj += sx[1][r] * v; }
    if (wsl == 0) ag -= bgj;
    if (wsl == 1) aj -= bgj;
    red[0][wsl][wrow] = ag; red[1][wsl][wrow] = aj;
  }
  __syncthreads();
  // p = ZT z = M^-1 t
  matvec(m_of, st, ma, mb);
  if (mq == 0) { sp[0][mr] = mr < tau ? ma : 0.0; sp[1][mr] = mr < tau ? mb : 0.0; }
  // x . k and x . t of the inner products of z_g, z_j
  if (wave >= W - 3) {
    const int k = wave - (W - 3);
    const int e0 = lane, e1 = lane + 64;
    double v;
    if (k == 1) v = sx[0][e0] * sk[1][e0] + sx[0][e1] * sk[1][e1] + sx[1][e0] * st[0][e0] + sx[1][e1] * st[0][e1];
    else { const int h = k >> 1; v = sx[h][e0] * (sk[h][e0] + st[h][e0]) + sx[h][e1] * (sk[h][e1] + st[h][e1]); }
    v = wsum(v);
    if (lane == 0) dots[3 + k] = v;
  }
  // the rows' dots with x while the products with M^-1 finish
  double da[4] = {0, 0, 0, 0};
  auto row_dot = [&](const double (*x)[TM], double& a, double& b) {
#pragma unroll
    for (int t = 0; t < CT; t++) {
      const int s = (lr + LPR * t) * 4;
      const double c0 = s < tau ? (double)c4[t].x : 0.0, c1 = s + 1 < tau ? (double)c4[t].y : 0.0;
      const double c2 = s + 2 < tau ? (double)c4[t].z : 0.0, c3 = s + 3 < tau ? (double)c4[t].w : 0.0;
      a += c0 * x[0][s] + c1 * x[0][s + 1] + c2 * x[0][s + 2] + c3 * x[0][s + 3];
      b += c0 * x[1][s] + c1 * x[1][s + 1] + c2 * x[1][s + 2] + c3 * x[1][s + 3];
    }
    a = sum8(a); b = sum8(b);
    if (LPR == 16) { a += dpp_get<0x140, 0xf>(a); b += dpp_get<0x140, 0xf>(b); }      // row_mirror: the other half row's sum
  };
  row_dot(sx, da[0], da[1]);
  __syncthreads();
  row_dot(sp, da[2], da[3]);
  // ---- the exact change of the objective (Case 3) and the acceptance test: the same numbers in every workgroup
  const double ngg = s_n0[0] - dots[0], njg = single ? 0.0 : s_n0[1] - dots[1], njj = s_n0[2] - dots[2];
  const bool bad1 = !(ngg < 0.0);                         // kept pivot: N_gg = -P_gg
  const double Dg = 1.0 / (bad1 ? -1.0 : ngg);
  const double M1 = Dg * njg;
  const double njjp = njj - njg * M1;                     // entering pivot after the first sweep: a Schur complement
  const bool bad2 = !single && !(njjp > 0.0);
  const double Dj = single ? 0.0 : 1.0 / (bad2 ? 1.0 : njjp);
  const double zgg = s_kk[0] - dots[3], zgj = single ? 0.0 : s_kk[1] - dots[4], zjj = single ? 0.0 : s_kk[2] - dots[5];
  // y1 = Dg z_g, y2 = Dj z_j', z_j' = z_j - M1 z_g
  const double zjjp = zjj - 2.0 * M1 * zgj + M1 * M1 * zgg;
  const double y11 = Dg * Dg * zgg, y12 = Dg * Dj * (zgj - M1 * zgg), y22 = Dj * Dj * zjjp;
  const double delta = -Dg * zgg - Dj * zjjp, obj = cin->obj;
  const bool notpd = bad1 || bad2 || cin->notpd;
  const bool ok = !notpd && (always || delta < -cin->rel_tol * obj);
  if (wg == 0 && tid == 0) {
    SearchCtrl c = *cin;
    const int it = c.iters;
    double m1 = s_v[0], m2 = s_2nd[0], x1 = s_v[W / 2], x2 = s_2nd[W / 2];
    for (int w = 1; w < W / 2; w++) { m1 = fmin(m1, s_v[w]); m2 = fmin(m2, s_2nd[w]); x1 = fmin(x1, s_v[W / 2 + w]); x2 = fmin(x2, s_2nd[W / 2 + w]); }
    c.gap_rem = isfinite(m2) ? fabs(m2 - m1) / fmax(fabs(m1), 1e-300) : INFINITY;
    c.gap_add = isfinite(x2) ? fabs(x1 - x2) / fmax(fabs(x1), 1e-300) : INFINITY;
    c.g_out = g; c.g_in = j; c.delta = delta; c.notpd = notpd ? 1 : 0; c.iters = it + 1; c.tau_inc = 0;
    if (ok) { c.obj = obj + delta; c.accepted += 1; c.tau = tau + npiv; } else c.done = 1;
    *cout = c;
    if (trace_out) trace_out[it] = g;
    if (trace_in) trace_in[it] = j;
    if (trace_gap) { trace_gap[2 * it] = (float)c.gap_rem; trace_gap[2 * it + 1] = (float)c.gap_add; }
    if (trace_obj) trace_obj[it] = ok ? obj + delta : obj;
  }
  if (!ok) { pass_on(-2, -1, -2, -1); return; }
  // ---- M^-1 bordered by g, then j
  if (mr < tau + npiv) {
    auto edge_g = [&](double x, double p) { return -x * Dg + p * M1 * Dj; };
    auto edge_j = [&](double p) { return -p * Dj; };
    const double xr = sx[0][mr], pr = sx[1][mr] - xr * M1;
    for (int u = own; u < MU && 2 * TPR * u < th; u += nwg) {
      const int c = 2 * TPR * u + 2 * mq;
      const double2 old = u == own ? mo : *reinterpret_cast<const double2*>(L.Minv + piece(u));
      double o[2] = {old.x, old.y};
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const int k = c + e, hi = max(mr, k);
        const double xs = sx[0][k], pc = sx[1][k] - xs * M1;
        if (hi < tau) o[e] += xr * xs * Dg + pr * pc * Dj;
        else if (hi == tau) o[e] = mr == k ? Dg + M1 * M1 * Dj : mr < k ? edge_g(xr, pr) : edge_g(xs, pc);
        else if (hi == tau + 1 && !single) o[e] = mr == k ? Dj : min(mr, k) == tau ? -M1 * Dj : edge_j(mr < k ? pr : pc);
        else o[e] = 0.0;
      }
      *reinterpret_cast<double2*>(L.Minv2 + piece(u)) = double2{o[0], o[1]};
    }
  }
  if (wg == nwg - 1 && tid < tau) {      // K_TT grows by the two pivots
    const double a = sk[0][tid], b = sk[1][tid];
    L.KT[tid * TM + tau] = a; L.KT[tau * TM + tid] = a;
    if (!single) { L.KT[tid * TM + tau + 1] = b; L.KT[(tau + 1) * TM + tid] = b; }
  }
  if (wg == nwg - 1 && tid == 0) {
    L.KT[tau * TM + tau] = s_kk[0];
    if (!single) { L.KT[tau * TM + tau + 1] = s_kk[1]; L.KT[(tau + 1) * TM + tau] = s_kk[1]; L.KT[(tau + 1) * TM + tau + 1] = s_kk[2]; }
  }
  // ---- the workgroup's rows: squared norms, diagonal, scores, the two new columns of C0
  const int rl = tid / LPR;
  double w1 = -red[0][lr][rl], w2 = -red[1][lr][rl];
  w1 = sum8(w1); w2 = sum8(w2);
  if (LPR == 16) { w1 += dpp_get<0x140, 0xf>(w1); w2 += dpp_get<0x140, 0xf>(w2); }
  if (lr == 0) {
    int kp = -1, sl = -1;
    double sc = 0.0;
    if (row < d1) {
      L.C0R[(int64_t)row * TM + tau] = n0g;
      if (!single) L.C0R[(int64_t)row * TM + tau + 1] = n0j;
      double r, dn;
      sl = slot0; kp = kp0;
      if (row == g) {
        r = y11 - 2.0 * M1 * y12 + M1 * M1 * y22;          // || -y1 + M1 y2 ||^2
        dn = -Dg - M1 * M1 * Dj;
        kp = 0; sl = PENDING;
        L.pos[row] = tau; L.Tidx[tau] = row; L.Jsg[tau] = -1.f; L.tslot[tau] = sg; kept[row] = 0;
      } else if (row == j) {
        r = y22; dn = -Dj;
        kp = 1; sl = PENDING;
        L.pos[row] = tau + 1; L.Tidx[tau + 1] = row; L.Jsg[tau + 1] = 1.f; L.tslot[tau + 1] = sj; kept[row] = 1;
      } else {
        // columns g, j of N and the products of the row of Z with y1, y2 (w = Z0 [y1 y2] from the products computed ahead, ZT [y1 y2])
        double c1, cj, zy1, zy2;
        if (ps >= 0) {
          const double sgn = (double)L.Jsg[ps], u1 = Dg * sp[0][ps];
          c1 = sgn * sx[0][ps]; cj = sgn * sx[1][ps];
          zy1 = sgn * u1; zy2 = sgn * Dj * (sp[1][ps] - njg * u1);
          sl = PENDING;
        } else {
          c1 = (double)n0g - da[0]; cj = (double)n0j - da[1];
          zy1 = Dg * (w1 - da[2]); zy2 = Dj * ((w2 - da[3]) - njg * zy1);
        }
        const double c2 = cj - c1 * M1;
        r = rho0 - 2.0 * c1 * zy1 + c1 * c1 * y11;           // after the reverse sweep on g
        const double zy2p = zy2 - c1 * y12;                  // (Z_i - c1 y1) . y2
        r += -2.0 * c2 * zy2p + c2 * c2 * y22;               // after the forward sweep on j
        if (r < 0.0) r = 0.0;
        dn = diag0 - c1 * c1 * Dg - c2 * c2 * Dj;
      }
      rho[row] = r; diag[row] = dn;
      sc = r / fabs(dn);
      score[row] = sc;
    }
    s_sc[rl] = sc; s_kp[rl] = kp; s_sl[rl] = sl;
  }
  __syncthreads();
  write_record<RPW>(L.rec2 + wg, s_sc, s_kp, s_sl, wg * RPW, wave, lane);
}

int swap_record_count(int64_t d1) { const int r = swap_rows_per_wg((int)d1); return (int)((d1 + r - 1) / r); }

hipError_t launch_lazy_swap(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, SearchCtrl* next, int always, int limit, int tau_most,
                            hipStream_t s, const SwapList& l, bool fetch_only) {
  if (l.n < 0 || l.n > LIST_MOST || (l.n > 0 && !l.out)) return hipErrorInvalidValue;
  // rows of more than 4096 columns: a workgroup for every compute unit, so that a fetch of few long rows is not left to a few of them (100
  // swaps, 72 pivots fetched: 1000 x 16384 8.4 ms without, 6.4 so; 300 x 8192, 60 swaps 3.0 and 2.4)
  const int nwg = swap_record_count(d.d1), grid = d.m > 4096 ? std::max(nwg, 256) : nwg;
#define OSSCAR_SWAP(NT, RPW)                                                                                                         \
  hipLaunchKernelGGL((lazy_swap_kernel<NT, RPW>), dim3(grid), dim3(NT), 0, s, L, t.N, t.Z, d.d1, d.m, t.ctrl, next, t.kept, t.gram, t.dblk, \
                     t.score, always, tau_most, l.out, l.in, l.n, l.step, limit, fetch_only ? 1 : 0, nwg, t.trace_out, t.trace_in, t.trace_gap, t.trace_obj)
  switch (swap_rows_per_wg(d.d1)) {
    case 32: OSSCAR_SWAP(512, 32); break;
    case 64: OSSCAR_SWAP(1024, 64); break;
    default: OSSCAR_SWAP(1024, 128); break;
  }
#undef OSSCAR_SWAP
  return hipGetLastError();
}

hipError_t launch_swap_records(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, bool refresh) {
  const int nwg = swap_record_count(d.d1), fr = refresh ? 1 : 0, words = RUN_SHARED_WORDS;
  uint64_t* shared = reinterpret_cast<uint64_t*>(L.run_shared);
  switch (swap_rows_per_wg(d.d1)) {
    case 32: hipLaunchKernelGGL(swap_records_kernel<32>, dim3(nwg), dim3(128), 0, s, L, d.d1, t.kept, t.score, t.gram, t.dblk, t.ctrl, fr, shared, words); break;
    case 64: hipLaunchKernelGGL(swap_records_kernel<64>, dim3(nwg), dim3(128), 0, s, L, d.d1, t.kept, t.score, t.gram, t.dblk, t.ctrl, fr, shared, words); break;
    default: hipLaunchKernelGGL(swap_records_kernel<128>, dim3(nwg), dim3(128), 0, s, L, d.d1, t.kept, t.score, t.gram, t.dblk, t.ctrl, fr, shared, words); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------- K and ZT
typedef double sw_d4 __attribute__((ext_vector_type(4)));
// K of the picked rows, Zc Zc^T with float64 sums, a workgroup per 16 x 16 tile of its lower triangle (n slots): every wave takes every
// W-th stretch of 16 columns on v_mfma_f64_16x16x4_f64, the waves' tiles are added in order.  Bound by the latency of a wave's loads.
constexpr int KW = 16;
__global__ __launch_bounds__(64 * KW) void cand_gram_kernel(LazyPtrs L, const float* __restrict__ Z0, int m) {
  __shared__ double part[KW][16][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  int I = 0, J = blockIdx.x;
  while (J > I) { J -= I + 1; I++; }
  const int ra = L.cand[I * 16 + lc], rb = L.cand[J * 16 + lc];
  const float *pa = Z0 + (int64_t)max(ra, 0) * m, *pb = Z0 + (int64_t)max(rb, 0) * m;
  sw_d4 acc = {0.0, 0.0, 0.0, 0.0};
  const int stretches = (m + 15) / 16;
  const bool vec = m % 4 == 0;
  for (int c0 = wave; c0 < stretches; c0 += 4 * KW) {        // four stretches requested at a time
    float a[4][4], b[4][4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int c = c0 + u * KW, k0 = c * 16;
      if (vec) {                                             // a lane's four values are one load; the order of the sum is free
        const int k = k0 + 4 * lr;
        const bool in = k < m;
        const float4 x = *reinterpret_cast<const float4*>(pa + (in ? k : 0)), y = *reinterpret_cast<const float4*>(pb + (in ? k : 0));
        const bool ia = in && ra >= 0, ib = in && rb >= 0;
        a[u][0] = ia ? x.x : 0.f; a[u][1] = ia ? x.y : 0.f; a[u][2] = ia ? x.z : 0.f; a[u][3] = ia ? x.w : 0.f;
        b[u][0] = ib ? y.x : 0.f; b[u][1] = ib ? y.y : 0.f; b[u][2] = ib ? y.z : 0.f; b[u][3] = ib ? y.w : 0.f;
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int k = k0 + 4 * e + lr;
          const bool in = k < m;
          const float x = pa[in ? k : 0], y = pb[in ? k : 0];
          a[u][e] = in && ra >= 0 ? x : 0.f; b[u][e] = in && rb >= 0 ? y : 0.f;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; u++)
#pragma unroll
      for (int e = 0; e < 4; e++) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[u][e], (double)b[u][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; r++) part[wave][4 * r + lr][lc] = acc[r];
  __syncthreads();
  if (tid < 256) {
    const int a = tid >> 4, b = tid & 15;
    double v = 0;
#pragma unroll
    for (int w = 0; w < KW; w++) v += part[w][a][b];
    const int i = I * 16 + a, j = J * 16 + b;
    if (j <= i) { L.K[i * KLD + j] = v; L.K[j * KLD + i] = v; }
  }
}
hipError_t launch_cand_gram(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, int ncand, hipStream_t s) {
  const int nt = (ncand + 15) / 16;
  if (nt > 0) hipLaunchKernelGGL(cand_gram_kernel, dim3(nt * (nt + 1) / 2), dim3(64 * KW), 0, s, L, t.Z, d.m);
  return hipGetLastError();
}

// ZT = M^-1 Z0[T, :] of a flush (zero from tau on), float64 and the float32 copy that the flush cuts into pieces.  A workgroup takes 16
// columns, its four waves 32 pending pivots each; the rows of M^-1 are read in pairs of columns, so the pivots' rows of Z0 are too.
__global__ __launch_bounds__(256) void zt_kernel(LazyPtrs L, const float* __restrict__ Z0, int m, const SearchCtrl* __restrict__ ctrl) {
  __shared__ int T[LAZY_TM];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
  const int tau = ctrl->tau + ctrl->tau_inc, col = blockIdx.x * 16 + lc, cc = min(col, m - 1);
  const double* Mi = L.Minv;
  if (tid < LAZY_TM) T[tid] = tid < tau ? L.Tidx[tid] : 0;
  __syncthreads();
  sw_d4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll 4
  for (int u = 0; u < LAZY_TM / 8; u++) {
    const int k = 8 * u + 2 * lr;
    const float z0 = Z0[(int64_t)T[k] * m + cc], z1 = Z0[(int64_t)T[k + 1] * m + cc];
    const double b0 = k < tau ? (double)z0 : 0.0, b1 = k + 1 < tau ? (double)z1 : 0.0;
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const double2 a = *reinterpret_cast<const double2*>(Mi + (wave * 32 + h * 16 + lc) * LAZY_TM + k);
      acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b0, acc[h], 0, 0, 0);
      acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b1, acc[h], 0, 0, 0);
    }
  }
  if (col >= m) return;
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = wave * 32 + h * 16 + 4 * r + lr;
      const double v = row < tau ? acc[h][r] : 0.0;
      L.ZT[(int64_t)row * m + col] = v; L.ZT32[(int64_t)row * m + col] = (float)v;
    }
}
hipError_t launch_zt(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s) {
  hipLaunchKernelGGL(zt_kernel, dim3((d.m + 15) / 16), dim3(256), 0, s, L, t.Z, d.m, t.ctrl);
  return hipGetLastError();
}

}  // namespace osscar
