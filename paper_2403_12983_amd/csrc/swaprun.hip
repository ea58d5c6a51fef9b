// Many swaps of the delayed-update search (q = 1) in one launch (swap.hip has the algebra of a swap and makes one of them per launch).
//
// The workgroups stay where they are from swap to swap.  M^-1 and L = ZT ZT^T are held in registers by every workgroup, which borders them for
// itself (with L in the place of K_TT a swap's x = M^-1 b and ZT z = M^-1 k - L b are one stage; with K_TT they are three in a row).  A
// workgroup's own rows of C0, their products with the pending pivots, norms, diagonals and scores are held by it alone.  What the workgroups
// have to tell one another is the best row of each side (a record of ten words) and the base columns of the pivots (C0).  Both go through
// memory past the XCDs' L2 caches: words of 32 bits beside the number of the exchange, so that a word tells by itself whether it has
// arrived, in two buffers that change place (a workgroup writes exchange e + 2 after it has read all of e + 1, which nobody sends before
// reading all of e).
// Bound by latency.  By cycle counts of the wave that sends the record (profiles/swap_kernels_pmc.md), at 8192 x 2048 (28672 x 512): from one record
// sent to the next pair picked 1.9 us (3.6), the pivots' rows and products 1.8 (2.4), the solve 1.4 (1.6), the rows' sums 1.25 (2.1), their
// norms and scores and the record 1.45 (2.1), barriers included; waves wait for 0.6 of their cycles.  A look at the records that comes too early
// costs more than it gains (the looks stand in the words' way), so every wave waits as long as its looks have lately had to.  A swap, launches
// and prologues included: 6.8 us at 8192 x 512, 8.7 at 16384 x 256, 10.9 - 11.3 at 28672 x 512 (a launch each: 11.5, 15, 20).
// A launch each pays for the records, M^-1 and the rows to come from memory each time, and for the launch.
//
// No workgroup waits for ever.  One that has waited `patience` gives up, and all of them then agree (arrived, verdict) whether the run
// counts: what a run leaves is written after that, so a run that does not count leaves the state as it was (what has two copies is copied:
// control block, records, M^-1, L), the runs enqueued behind it make no swap, and the host makes them a launch each.  That happens where
// other work keeps some of the workgroups from starting.
// GIVEN: the pairs stand in a list, nothing has to be agreed on, and no workgroup waits for another.
#include "internal.h"
#include "lazy_device.h"
#include "wave.h"
#include <algorithm>

namespace osscar {

constexpr int RT = 512;                     // threads: 32 groups of 16 lanes, a group four rows of M^-1, a lane eight of their columns
constexpr int KROW = LAZY_NC + LAZY_NS;     // row length of K
constexpr int WORDS = RUN_WORDS;            // of a record's side: best value (2), row and slot, second best value (2)
// cycles from a swap's last barrier to a wave's first look at the next records: at first; less after a look that found them, more after one
// that came too early (9.5 us a swap with looks at once, 6.9 so)
constexpr int HOLD_START = 2000, HOLD_LESS = 16, HOLD_MORE = 256, HOLD_MOST = 16384;
constexpr int PEND = 1 << 30;               // flag in a record's slot: the row is a pending pivot
struct RunShared { uint64_t word[2][2 * WORDS][RUN_WGS]; int32_t arrived[RUN_MOST], verdict[RUN_MOST]; };
static_assert(sizeof(RunShared) == RUN_SHARED_WORDS * 8, "as the workspace has room for");
static_assert(LAZY_TM == 128, "four stretches of 32 columns");

typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ T seen(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void show(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ double lesser(double a, double b) { return b < a ? b : a; }
// the first lane with the least value among those with i >= 0 (lane 0 if there is none): lanes are in the order of the rows, and of equal values
// the lowest row is meant
__device__ __forceinline__ int first_best(double v, int i) {
  double m = i >= 0 ? v : INFINITY;
  m = lesser(m, dpp_get_or<0xb1, 0xf>(m, INFINITY)); m = lesser(m, dpp_get_or<0x4e, 0xf>(m, INFINITY));
  m = lesser(m, dpp_get_or<0x124, 0xf>(m, INFINITY)); m = lesser(m, dpp_get_or<0x128, 0xf>(m, INFINITY));
  m = lesser(m, dpp_get_or<0x142, 0xa>(m, INFINITY)); m = lesser(m, dpp_get_or<0x143, 0xc>(m, INFINITY));
  m = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(m), 63), __builtin_amdgcn_readlane(__double2loint(m), 63));
  const uint64_t who = __ballot(i >= 0 && v == m), any = __ballot(i >= 0);
  return who ? (int)__builtin_ctzll(who) : any ? (int)__builtin_ctzll(any) : 0;
}
__device__ __forceinline__ double from_lane(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sums over the 16 lanes of a group, of 2 R values v[h][i] (h: vector, i: row): lane l is left with (h, i) = (bit 3, 2 bit 2 + bit 0) for
// R = 4, (bit 3, bit 2) for 2, (bit 3, 0) for 1.
template <int R>
__device__ __forceinline__ double group_sums(const double (&v)[2][R], int l) {
  const bool b3 = l & 8, b2 = l & 4, b0 = l & 1;
  double a[R];
#pragma unroll
  for (int i = 0; i < R; i++) {
    const double keep = b3 ? v[1][i] : v[0][i], give = b3 ? v[0][i] : v[1][i];
    a[i] = keep + dpp_get<0x140, 0xf>(give);           // row_mirror: lane 15 - l
  }
  double t;
  if constexpr (R == 4) {
    double c[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const double keep = b2 ? a[2 + i] : a[i], give = b2 ? a[i] : a[2 + i];
      c[i] = keep + dpp_get<0x141, 0xf>(give);         // row_half_mirror
    }
    const double keep = b0 ? c[1] : c[0], give = b0 ? c[0] : c[1];
    t = keep + dpp_get<0xb1, 0xf>(give);
  } else if constexpr (R == 2) {
    const double keep = b2 ? a[1] : a[0], give = b2 ? a[0] : a[1];
    t = keep + dpp_get<0x141, 0xf>(give);
    t += dpp_get<0xb1, 0xf>(t);
  } else {
    t = a[0] + dpp_get<0x141, 0xf>(a[0]);
    t += dpp_get<0xb1, 0xf>(t);
  }
  return t + dpp_get<0x4e, 0xf>(t);
}
template <int R> __device__ __forceinline__ int sum_row(int l) { return R == 4 ? ((l >> 1) & 2) | (l & 1) : R == 2 ? (l >> 2) & 1 : 0; }
// one of the lanes that are left with a sum
template <int R> __device__ __forceinline__ bool sum_lane(int l) { return R == 4 ? !(l & 2) : R == 2 ? !(l & 3) : !(l & 7); }

// RPW rows per workgroup as in swap.hip (the records of both are the same ones).  Workgroup of the run number `run` since the shared words were cleared.
struct RunArgs {
  // from swap to swap
  const float* N0; const double *GbT, *K; float* C0R; RunShared* sh;
  int d1, nwg, limit, run, list_n, always; uint32_t patience;
  int32_t *trace_out, *trace_in; float* trace_gap; double* trace_obj;
  // before the first and after the last one
  const SearchCtrl* cin; SearchCtrl* cout;
  int32_t *kept, *pos, *Tidx, *tslot; const int32_t* cslot; float* Jsg; double *rho, *diag, *score;
  const double *Minv, *LL; double *Minv2, *LL2, *KT; const SwapRec* rec; SwapRec* rec2;
  const int32_t *list_g, *list_j; int list_step;
};
typedef const __attribute__((address_space(4))) RunArgs* RunArgsPtr;
// the arguments, to be read again here (kept in registers through the swaps they left none for the swaps)
__device__ __forceinline__ RunArgsPtr args_again() {
  RunArgsPtr p = (RunArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

template <int RPW, bool GIVEN>
__global__ __launch_bounds__(RT) void swap_run_kernel(const RunArgs A) {
  constexpr int TM = LAZY_TM, R = RPW / 32, RW = 6, RWAVES = (RPW + 63) / 64;      // rows of a group; waves of the row threads: RW .. (they and the two before
                                                                                 // them hold the rows of M^-1 that are used last)
  constexpr bool C_LDS = R >= 2;                                  // C0 of several rows, and of four the products' last stretch,
  constexpr int GV = R == 4 ? 3 : 4;                              // are in shared memory: the registers do not hold them
  __shared__ double s_v[2][8], s_2nd[8];      // (the gaps are taken while other waves are at the next pick)
  __shared__ int s_i[8], s_s[8], s_T[TM], s_slot[TM], s_flag, s_late;
  __shared__ __attribute__((aligned(16))) double sb[2][TM], sk[2][TM], sx[2][TM], sp[2][TM], sa[4][TM];
  __shared__ double s_kk[3], s_row[4][RPW], s_new[2][RPW], s_half[2][2];
  __shared__ float s_n0[3], s_c[2][RPW];
  __shared__ double s_rho[RPW], s_diag[RPW], s_score[RPW];      // the workgroup's rows
  __shared__ int s_kept[RPW], s_pos[RPW], s_own[RPW];
  __shared__ signed char s_sign[TM];
  __shared__ int s_hrow[2], s_hslot[2], s_list[GIVEN ? 4 : 1][GIVEN ? 64 : 1];
  __shared__ SwapRec s_rec;
  // of the swap: its scalars; of the run: what the control block is left with
  __shared__ struct { double Dg, Dj, M1, njg, zgg, zgj, zjj; int bad; } s_q;
  __shared__ struct { double delta, gap_rem, gap_add; } s_run;
  __shared__ double s_obj[2];      // before and after the swap
  __shared__ f2 s_c0[C_LDS ? 4 * R * RT : 1];
  __shared__ d2 s_gb[GV < 4 ? R * RT : 1];
  const int wg = blockIdx.x;
  // what a thread is.  (Asked again for every swap and at the end: kept, these and the addresses that follow from them go to scratch memory.)
#define OSSCAR_RUN_THREAD                                                                                                        \
  int tid = threadIdx.x;                                                                                                         \
  asm volatile("" : "+v"(tid));                                                                                                  \
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 15, rq = tid >> 4, rt = tid & 255;        \
  const int side = wave >> 2;                                                                                                    \
  const bool row_thread = wave >= RW && tid - 64 * RW < RPW;      /* 64 RW .. 64 RW + RPW: a row each */                          \
  const int lrow = row_thread ? tid - 64 * RW : 0, row = wg * RPW + lrow, rc = min(row, d1 - 1);                                  \
  const bool has_row = row_thread && row < d1;                                                                                   \
  (void)lane; (void)l; (void)rq; (void)rt; (void)side; (void)rc; (void)has_row
  RunArgsPtr P = args_again();
  const float* const N0 = A.N0;
  const int d1 = P->d1, nwg = P->nwg, run = P->run;
  OSSCAR_RUN_THREAD;
  int limit = P->cin->stalled ? 0 : P->limit;      // (a launch before this one was given up: the host goes on)
  // ---- the state as the last launch left it
  int tau = P->cin->tau, iters = P->cin->iters, done = P->cin->done, pause = P->cin->pause, notpd = P->cin->notpd, accepted = 0;
  const int spare = P->cin->spare, tau_start = tau;
  if (done | pause) limit = iters;
  if (tid < TM) { const bool in = tid < tau; s_T[tid] = in ? P->Tidx[tid] : 0; s_slot[tid] = in ? P->tslot[tid] : 0; s_sign[tid] = in && P->Jsg[tid] > 0.f ? 1 : -1; }
  if (tid == 0) {
    s_flag = 0; s_late = 0; s_rec = P->rec[wg]; s_obj[iters & 1] = P->cin->obj;
    s_run.delta = P->cin->delta; s_run.gap_rem = P->cin->gap_rem; s_run.gap_add = P->cin->gap_add;
  }
  d2 mv[4][4], lv[4][4];      // M^-1 and ZT ZT^T: rows 4 rq + i, columns 32 v + 2 l and the next
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int v = 0; v < 4; v++) { mv[i][v] = d2{0.0, 0.0}; lv[i][v] = d2{0.0, 0.0}; }
  if (tau > 0) {      // (loads without conditions: one under a condition of its own is waited for where it ends)
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int at = (4 * rq + i) * TM + 32 * v + 2 * l;
        mv[i][v] = *reinterpret_cast<const d2*>(P->Minv + at); lv[i][v] = *reinterpret_cast<const d2*>(P->LL + at);
      }
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int v = 0; v < 4; v++)
        if (4 * rq + i >= tau || 32 * v + 2 * l >= tau) { mv[i][v] = d2{0.0, 0.0}; lv[i][v] = d2{0.0, 0.0}; }      // not defined there; tau is even
  }
  __syncthreads();
  d2 gb[R][GV];      // products of the group's rows with the pending pivots
  f2 c4[C_LDS ? 1 : R][4];
#pragma unroll
  for (int i = 0; i < R; i++)
#pragma unroll
    for (int v = 0; v < 4; v++) {
      if (v < GV) gb[i][v] = d2{0.0, 0.0}; else s_gb[i * RT + tid] = d2{0.0, 0.0};
      if constexpr (C_LDS) s_c0[(i * 4 + v) * RT + tid] = f2{0.f, 0.f}; else c4[i][v] = f2{0.f, 0.f};
    }
  if (tau > 0) {
#pragma unroll
    for (int i = 0; i < R; i++) {
      const int r = min(wg * RPW + R * rq + i, d1 - 1);
      f2 f[4];
      d2 y[4];
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int c = 32 * v + 2 * l;
        y[v] = d2{P->GbT[(int64_t)s_slot[c] * d1 + r], P->GbT[(int64_t)s_slot[c + 1] * d1 + r]};
        f[v] = *reinterpret_cast<const f2*>(P->C0R + (int64_t)r * TM + c);
      }
#pragma unroll
      for (int v = 0; v < 4; v++) {
        if (32 * v + 2 * l >= tau) { y[v] = d2{0.0, 0.0}; f[v] = f2{0.f, 0.f}; }
        if (v < GV) gb[i][v] = y[v]; else s_gb[i * RT + tid] = y[v];
        if constexpr (C_LDS) s_c0[(i * 4 + v) * RT + tid] = f[v]; else c4[i][v] = f[v];
      }
    }
  }
  if (row_thread) {
    s_rho[lrow] = P->rho[rc]; s_diag[lrow] = P->diag[rc]; s_score[lrow] = P->score[rc];
    s_kept[lrow] = has_row ? (P->kept[rc] != 0) : -1; s_pos[lrow] = P->pos[rc]; s_own[lrow] = P->cslot[rc];
  }
  if constexpr (GIVEN) {      // the list with its rows' slots
    if (tid < 64) {
      const int at = min(lane, P->list_n - 1) * P->list_step, lg = P->list_g[at], lj = P->list_j[at];
      const bool in = lg >= 0 && lg < d1 && lj >= 0 && lj < d1;
      s_list[0][lane] = in ? lg : -1; s_list[1][lane] = in ? lj : -1;
      s_list[2][lane] = in ? P->cslot[lg] : -1; s_list[3][lane] = in ? P->cslot[lj] : -1;
    }
    __syncthreads();
  }
  int exchanges = 0, g_out = P->cin->g_out, g_in = P->cin->g_in;
  bool stalled = false, swapped = false, waited = false;
  const double rel_tol = P->cin->rel_tol;
  int hold = HOLD_START;
  uint64_t sent = 0;

  while (iters < limit && !done && !pause) {
    OSSCAR_RUN_THREAD;
    auto c_of = [&](int i, int v) -> f2 { if constexpr (C_LDS) return s_c0[(i * 4 + v) * RT + tid]; else return c4[i][v]; };
    int g, j, sg, sj;
    int pick_g = -1, pick_j = -1;
    double v1 = INFINITY, v2 = INFINITY;
    int i1 = -1, sl1 = -1;
    if constexpr (!GIVEN) {
      // ---- the records: the last launch's, then the other workgroups' as they arrive
      if (exchanges == 0) {
        const SwapRec* rp = args_again()->rec + min(rt, nwg - 1);
        v1 = rp->best[side]; v2 = rp->second[side]; i1 = rp->row[side]; sl1 = rp->slot[side];
      } else {
        const uint32_t tag = (uint32_t)(run * 256 + exchanges);
        const uint64_t* w = A.sh->word[exchanges & 1][side * WORDS] + min(rt, nwg - 1);
        uint64_t x[3], t0 = 0;
        waited = true;
        while (__builtin_readcyclecounter() - sent < (uint64_t)hold) __builtin_amdgcn_s_sleep(1);
        bool first = true;
        while (true) {
          bool ok = true;
#pragma unroll
          for (int k = 0; k < 3; k++) x[k] = seen(w + k * RUN_WGS);
#pragma unroll
          for (int k = 0; k < 3; k++) ok = ok && (uint32_t)(x[k] >> 32) == tag;
          if (__all(ok)) { if (first) hold = max(hold - HOLD_LESS, 0); break; }
          if (first) hold = min(hold + HOLD_MORE, HOLD_MOST);
          first = false;
          const uint64_t now = __builtin_amdgcn_s_memrealtime();
          if (t0 == 0) t0 = now;
          if (now - t0 >= args_again()->patience || seen(&A.sh->verdict[run]) != 0) { s_flag = 1; break; }
        }
        v1 = __hiloint2double((int)(uint32_t)x[0], (int)(uint32_t)x[1]);
        const int id = (int)(uint32_t)x[2];
        i1 = (id & (1 << 30)) ? (id & 0xffff) : -1;
        sl1 = (id & (1 << 29)) ? PEND : ((id >> 16) & 0x1ff) - 1;
      }
      if (rt >= nwg) { v1 = INFINITY; v2 = INFINITY; i1 = -1; sl1 = -1; }
      // ---- pick: waves 0 - 3 hold the leaving side's records, the others the entering side's
      if (lane == first_best(v1, i1)) { s_v[exchanges & 1][wave] = v1; s_i[wave] = i1; s_s[wave] = sl1; }
      __syncthreads();
      if (s_flag) { stalled = true; break; }
      const double qv = s_v[exchanges & 1][lane & 7];
      const int qi = s_i[lane & 7], qs = s_s[lane & 7];
      double mg = qi >= 0 ? qv : INFINITY;
      mg = lesser(mg, dpp_get<0xb1, 0xf>(mg)); mg = lesser(mg, dpp_get<0x4e, 0xf>(mg));      // of lanes 0 - 3 and 4 - 7
      const uint64_t best = __ballot(qi >= 0 && qv == mg);
      const int at_g = (best & 0xf) ? (int)__builtin_ctzll(best & 0xf) : 0, at_j = (best & 0xf0) ? (int)__builtin_ctzll(best & 0xf0) : 4;
      g = (best & 0xf) ? __builtin_amdgcn_readlane(qi, at_g) : -1; j = (best & 0xf0) ? __builtin_amdgcn_readlane(qi, at_j) : -1;
      sg = __builtin_amdgcn_readlane(qs, at_g); sj = __builtin_amdgcn_readlane(qs, at_j);
      pick_g = g; pick_j = j;
    } else {
      const int entry = __builtin_amdgcn_readfirstlane(min(max(iters - (A.limit - A.list_n), 0), A.list_n - 1));
      g = s_list[0][entry]; j = s_list[1][entry]; sg = s_list[2][entry]; sj = s_list[3][entry];
      const int T0 = lane < tau ? s_T[lane] : -1, T1 = lane + 64 < tau ? s_T[lane + 64] : -1;
      if (__any(T0 == g || T1 == g)) sg = PEND;
      if (__any(T0 == j || T1 == j)) sj = PEND;
    }
    g = __builtin_amdgcn_readfirstlane(g); j = __builtin_amdgcn_readfirstlane(j);
    sg = __builtin_amdgcn_readfirstlane(sg); sj = __builtin_amdgcn_readfirstlane(sj);
    if (g < 0 || j < 0) { done = 1; g_out = -1; g_in = -1; break; }
    const bool hit = sg >= 0 && sg < LAZY_NC + spare && sj >= 0 && sj < LAZY_NC + spare;
    if (sg == PEND || sj == PEND || tau + 2 > TM) { pause = 1; break; }
    if (!hit) break;      // the next launch fetches its products (and pauses if there is no slot)
    const int th = min(TM, (tau + 2 + 31) & ~31);
    // ---- everything that depends on the pick, in one round trip.  Threads 0 - 255: the pivots' rows of C0 and of K; 256 - 258: the
    // pivots' own; from 384 on: the workgroup's rows.
    const int bc = tid & (TM - 1), bh = (tid >> 7) & 1;
    {
      const int e2 = min(tid & 3, 2), er = e2 == 0 ? g : j, ec = e2 == 2 ? j : g;      // (g, g), (j, g), (j, j)
      const int pr = bh ? j : g, tc = s_T[bc];
      auto nsym = [&](int a, int b) { return N0 + (a >= b ? (int64_t)a * d1 + b : (int64_t)b * d1 + a); };
      const float* pa = tid < 256 ? (GIVEN ? nsym(pr, tc) : A.C0R + (int64_t)pr * TM + bc) : tid < 384 ? nsym(er, ec) : nsym(rc, g);
      const float* pb = nsym(rc, j);
      const double* pc = tid < 256 ? A.K + (bh ? sj : sg) * KROW + s_slot[bc] : tid < 384 ? A.K + (e2 == 0 ? sg : sj) * KROW + (e2 == 2 ? sj : sg) : A.GbT + (int64_t)sg * d1 + rc;
      const double* pd = A.GbT + (int64_t)sj * d1 + rc;
      const float a = GIVEN ? *pa : seen(pa), b = *pb;
      const double c = *pc, d = *pd;
      if (tid < 256) { const bool use = bc < tau; sb[bh][bc] = use ? (double)a : 0.0; sk[bh][bc] = use ? c : 0.0; }
      else if (tid < 259) { s_n0[tid - 256] = a; s_kk[tid - 256] = c; }
      else if (row_thread) {
        s_c[0][lrow] = a; s_c[1][lrow] = b; s_new[0][lrow] = c; s_new[1][lrow] = d;
        if (has_row) show(reinterpret_cast<uint64_t*>(A.C0R + (int64_t)row * TM + tau), ((uint64_t)__float_as_uint(b) << 32) | __float_as_uint(a));
      }
      if constexpr (!GIVEN) {
        if (wg == 0) {      // second-best values: every record's best unless it is the pick
          if (exchanges > 0) {      // (sent behind the others' first words, which are here; should they be late by `patience` the run does not count)
            const uint64_t* w = A.sh->word[exchanges & 1][side * WORDS + 3] + min(rt, nwg - 1);
            uint64_t hi, lo, t0 = 0;
            while (true) {
              hi = seen(w); lo = seen(w + RUN_WGS);
              if (__all((uint32_t)(hi >> 32) == (uint32_t)(run * 256 + exchanges) && (uint32_t)(lo >> 32) == (uint32_t)(run * 256 + exchanges))) break;
              const uint64_t now = __builtin_amdgcn_s_memrealtime();
              if (t0 == 0) t0 = now;
              if (now - t0 >= args_again()->patience) { s_late = 1; break; }
            }
            v2 = rt < nwg ? __hiloint2double((int)(uint32_t)hi, (int)(uint32_t)lo) : INFINITY;
          }
          const double sec = wave_min(i1 >= 0 && i1 != (side ? pick_j : pick_g) ? v1 : v2);
          if (lane == 63) s_2nd[wave] = sec;
        }
      }
    }
    __syncthreads();
    const bool rows_in = __builtin_amdgcn_readfirstlane(4 * rq) < th;      // 16 rows a wave: all of them or none
    const int oh = l >> 3, orow = 4 * rq + sum_row<4>(l);
    const bool owner = sum_lane<4>(l);
    // x = M^-1 b, p = ZT z = M^-1 k - (ZT ZT^T) b (z = Z0[g] - b^T ZT, ZT Z0[g]^T = M^-1 k): one stage (as t = k - K_TT x, p = M^-1 t they
    // are three in a row)
    if (rows_in) {
      double acc[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}}, acp[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
      for (int v = 0; v < 4; v++) {
        if (32 * v < th) {
          const int c = 32 * v + 2 * l;
          const d2 bg = *reinterpret_cast<const d2*>(&sb[0][c]), bj = *reinterpret_cast<const d2*>(&sb[1][c]);
          const d2 kg = *reinterpret_cast<const d2*>(&sk[0][c]), kj = *reinterpret_cast<const d2*>(&sk[1][c]);
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const d2 m = mv[i][v], n = lv[i][v];
            acc[0][i] += m.x * bg.x + m.y * bg.y; acc[1][i] += m.x * bj.x + m.y * bj.y;
            acp[0][i] += (m.x * kg.x + m.y * kg.y) - (n.x * bg.x + n.y * bg.y); acp[1][i] += (m.x * kj.x + m.y * kj.y) - (n.x * bj.x + n.y * bj.y);
          }
        }
      }
      const double x = group_sums<4>(acc, l), p = group_sums<4>(acp, l);
      if (owner) { sx[oh][orow] = x; sp[oh][orow] = p; }
    } else if (owner) { sx[oh][orow] = 0.0; sp[oh][orow] = 0.0; }
    __syncthreads();
    // the pivots' own: two waves
    if (wave == 4 || wave == 5) {
      __builtin_amdgcn_s_setprio(2);
      const int e0 = lane, e1 = lane + 64;
      const double bg0 = sb[0][e0], bg1 = sb[0][e1], bj0 = sb[1][e0], bj1 = sb[1][e1];
      const double xg0 = sx[0][e0], xg1 = sx[0][e1], xj0 = sx[1][e0], xj1 = sx[1][e1], pg0 = sp[0][e0], pg1 = sp[0][e1], pj0 = sp[1][e0], pj1 = sp[1][e1];
      if (wave == 4) {
        const double gg = wsum(bg0 * xg0 + bg1 * xg1), jg = wsum(bj0 * xg0 + bj1 * xg1), jj = wsum(bj0 * xj0 + bj1 * xj1);
        const double ngg = (double)s_n0[0] - gg, njg = (double)s_n0[1] - jg, njj = (double)s_n0[2] - jj;
        const bool bad1 = !(ngg < 0.0);                         // kept pivot: N_gg = -P_gg
        const double Dg = 1.0 / (bad1 ? -1.0 : ngg);
        const double M1 = Dg * njg;
        const double njjp = njj - njg * M1;                     // entering pivot after the first sweep: a Schur complement
        const bool bad2 = !(njjp > 0.0);
        const double Dj = 1.0 / (bad2 ? 1.0 : njjp);
        // M^-1 bordered by g, then j: M' = M + Dg a a^T + Dj b b^T, a = (x_g, -1, 0), b = (x_j - M1 x_g, M1, -1), and ZT' = ZT - a y1^T - b y2^T;
        // u1 = ZT y1, u2 = ZT y2
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const int k = lane + 64 * h;
          const double xg = h ? xg1 : xg0, xj = h ? xj1 : xj0, pg = h ? pg1 : pg0, pj = h ? pj1 : pj0;
          sa[0][k] = k == tau ? -1.0 : xg;      // (x and p are zero from tau on)
          sa[1][k] = k == tau ? M1 : k == tau + 1 ? -1.0 : xj - xg * M1;
          sa[2][k] = Dg * pg; sa[3][k] = Dj * (pj - M1 * pg);
        }
        if (lane == 0) { s_q.Dg = Dg; s_q.Dj = Dj; s_q.M1 = M1; s_q.njg = njg; s_q.bad = bad1 || bad2; }
        if (lane == 1) { s_T[tau] = g; s_slot[tau] = sg; s_T[tau + 1] = j; s_slot[tau + 1] = sj; s_sign[tau] = -1; s_sign[tau + 1] = 1; }
      } else {
        // z_a . z_b = K_ab - b_a . p_b - x_b . k_a
        const double kg0 = sk[0][e0], kg1 = sk[0][e1], kj0 = sk[1][e0], kj1 = sk[1][e1];
        const double gg = wsum(bg0 * pg0 + bg1 * pg1 + xg0 * kg0 + xg1 * kg1), gj = wsum(bg0 * pj0 + bg1 * pj1 + xj0 * kg0 + xj1 * kg1);
        const double jj = wsum(bj0 * pj0 + bj1 * pj1 + xj0 * kj0 + xj1 * kj1);
        if (lane == 0) { s_q.zgg = s_kk[0] - gg; s_q.zgj = s_kk[1] - gj; s_q.zjj = s_kk[2] - jj; }
      }
      __builtin_amdgcn_s_setprio(0);
    }
    // the rows' sums over the pending pivots: products with x (and C0 with p), C0 with x
    {
      double w[2][R], c[2][R];
#pragma unroll
      for (int i = 0; i < R; i++) { w[0][i] = 0; w[1][i] = 0; c[0][i] = 0; c[1][i] = 0; }
#pragma unroll
      for (int v = 0; v < 4; v++) {
        if (32 * v < th) {
          const int at = 32 * v + 2 * l;
          const d2 xg = *reinterpret_cast<const d2*>(&sx[0][at]), xj = *reinterpret_cast<const d2*>(&sx[1][at]);
          const d2 pg = *reinterpret_cast<const d2*>(&sp[0][at]), pj = *reinterpret_cast<const d2*>(&sp[1][at]);
#pragma unroll
          for (int i = 0; i < R; i++) {
            d2 y;
            if (v < GV) y = gb[i][v]; else y = s_gb[i * RT + tid];
            const f2 f = c_of(i, v);
            const double f0 = (double)f.x, f1 = (double)f.y;
            c[0][i] += f0 * xg.x + f1 * xg.y; c[1][i] += f0 * xj.x + f1 * xj.y;
            w[0][i] += (y.x * xg.x + y.y * xg.y) + (f0 * pg.x + f1 * pg.y); w[1][i] += (y.x * xj.x + y.y * xj.y) + (f0 * pj.x + f1 * pj.y);
          }
        }
      }
      const double ws = group_sums<R>(w, l), cs = group_sums<R>(c, l);
      if (sum_lane<R>(l)) { const int k = R * rq + sum_row<R>(l); s_row[oh][k] = s_new[oh][k] - ws; s_row[2 + oh][k] = cs; }
    }
    // what the rows need besides: of a pending row (row ps of T) columns g, j of N are multiples of x, and its products of p
    int kp = -1, ps = -1, own = -1;
    double rho_r = 0.0, diag_r = 1.0, cg = 0.0, cj = 0.0, qg = 0.0, qj = 0.0;
    if (wave >= RW && wave < RW + RWAVES) {
      if (has_row) { kp = s_kept[lrow]; ps = s_pos[lrow]; own = s_own[lrow]; }
      rho_r = s_rho[lrow]; diag_r = s_diag[lrow];
      const int pc = max(ps, 0);
      const double sgn = (double)s_sign[pc], xg = sgn * sx[0][pc], xj = sgn * sx[1][pc], pg = sgn * sp[0][pc], pj = sgn * sp[1][pc];
      const double fg = (double)s_c[0][lrow], fj = (double)s_c[1][lrow];
      cg = ps >= 0 ? xg : fg; cj = ps >= 0 ? xj : fj; qg = pg; qj = pj;
    }
    __syncthreads();
    // ---- the exact change of the objective (Case 3) and the acceptance test: the same numbers in every workgroup
    const double Dg = s_q.Dg, Dj = s_q.Dj, M1 = s_q.M1, njg = s_q.njg, zgg = s_q.zgg, zgj = s_q.zgj, zjj = s_q.zjj;
    // y1 = Dg z_g, y2 = Dj z_j', z_j' = z_j - M1 z_g
    const double zjjp = zjj - 2.0 * M1 * zgj + M1 * M1 * zgg;
    const double y11 = Dg * Dg * zgg, y12 = Dg * Dj * (zgj - M1 * zgg), y22 = Dj * Dj * zjjp;
    const double delta = -Dg * zgg - Dj * zjjp, obj = s_obj[iters & 1];
    notpd |= s_q.bad;
    const bool ok = __builtin_amdgcn_readfirstlane(!notpd && (A.always || delta < -rel_tol * obj));
    if (wave == 5 && lane == 0) {
      s_obj[(iters + 1) & 1] = ok ? obj + delta : obj;
      s_run.delta = delta;
      if (wg == 0) {
        double gap_rem = INFINITY, gap_add = INFINITY;
        if constexpr (!GIVEN) {
          const double* sv = s_v[exchanges & 1];
          double m1 = sv[0], m2 = s_2nd[0], x1 = sv[4], x2 = s_2nd[4];
          for (int w = 1; w < 4; w++) { m1 = fmin(m1, sv[w]); m2 = fmin(m2, s_2nd[w]); x1 = fmin(x1, sv[4 + w]); x2 = fmin(x2, s_2nd[4 + w]); }
          gap_rem = isfinite(m2) ? fabs(m2 - m1) / fmax(fabs(m1), 1e-300) : INFINITY;
          gap_add = isfinite(x2) ? fabs(x1 - x2) / fmax(fabs(x1), 1e-300) : INFINITY;
        }
        s_run.gap_rem = gap_rem; s_run.gap_add = gap_add;
        RunArgsPtr Q = args_again();
        if (Q->trace_out) Q->trace_out[iters] = g;
        if (Q->trace_in) Q->trace_in[iters] = j;
        if (Q->trace_gap) { Q->trace_gap[2 * iters] = (float)gap_rem; Q->trace_gap[2 * iters + 1] = (float)gap_add; }
        if (Q->trace_obj) Q->trace_obj[iters] = ok ? obj + delta : obj;
      }
    }
    g_out = g; g_in = j;
    iters++;
    if (!ok) { done = 1; break; }
    accepted++;
    // ---- the workgroup's rows: squared norms, diagonal, scores
    double bv[2] = {INFINITY, INFINITY}, b2[2] = {INFINITY, INFINITY};      // best and second best of each side among the wave's rows
    int br[2] = {-1, -1}, bs[2] = {-1, -1};
    if (wave >= RW && wave < RW + RWAVES) {
      __builtin_amdgcn_s_setprio(2);
      double sc = 0.0, r, dn;
      {
        // columns g, j of N and the products of the row of Z with y1, y2 (w = Z0 [y1 y2] from the products computed ahead, ZT [y1 y2])
        const double tg = s_row[0][lrow], tj = s_row[1][lrow], hg = s_row[2][lrow], hj = s_row[3][lrow];
        const bool in_t = ps >= 0;
        const double c1 = in_t ? cg : cg - hg, c1j = in_t ? cj : cj - hj;
        const double zy1 = Dg * (in_t ? qg : tg), zy2 = Dj * ((in_t ? qj : tj) - njg * zy1);
        const double c2 = c1j - c1 * M1;
        r = rho_r - 2.0 * c1 * zy1 + c1 * c1 * y11;          // after the reverse sweep on g
        const double zy2p = zy2 - c1 * y12;                  // (Z_i - c1 y1) . y2
        r += -2.0 * c2 * zy2p + c2 * c2 * y22;               // after the forward sweep on j
        if (r < 0.0) r = 0.0;
        dn = diag_r - c1 * c1 * Dg - c2 * c2 * Dj;
      }
      if (has_row) {
        if (row == g) {
          r = y11 - 2.0 * M1 * y12 + M1 * M1 * y22;          // || -y1 + M1 y2 ||^2
          dn = -Dg - M1 * M1 * Dj;
          kp = 0; ps = tau;
          s_kept[lrow] = kp; s_pos[lrow] = ps;
        } else if (row == j) {
          r = y22; dn = -Dj;
          kp = 1; ps = tau + 1;
          s_kept[lrow] = kp; s_pos[lrow] = ps;
        }
        sc = r / fabs(dn);
        s_rho[lrow] = r; s_diag[lrow] = dn; s_score[lrow] = sc;
      }
      const int sl = ps >= 0 ? PEND : own;
      const bool live = lane < RPW;
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const bool has = live && kp == 1 - h && sc == sc;      // (no record of a NaN, as in write_record)
        const double v = h == 0 ? sc : -sc;
        const int at = first_best(v, has ? row : -1);
        const bool some = __any(has);
        br[h] = some ? __builtin_amdgcn_readlane(row, at) : -1;
        bv[h] = some ? from_lane(v, at) : INFINITY;
        bs[h] = some ? __builtin_amdgcn_readlane(sl, at) : -1;
        b2[h] = has && lane != at ? v : INFINITY;      // the lane's; their least value follows where it is wanted
      }
      if constexpr (RWAVES == 2) {      // the second wave hands its half to the first
        const double m2[2] = {from_lane(wave_min(b2[0]), 63), from_lane(wave_min(b2[1]), 63)};
        if (wave == RW + 1 && lane < 2) { s_half[lane][0] = lane ? bv[1] : bv[0]; s_half[lane][1] = lane ? m2[1] : m2[0]; s_hrow[lane] = lane ? br[1] : br[0]; s_hslot[lane] = lane ? bs[1] : bs[0]; }
        __builtin_amdgcn_s_waitcnt(0);      // C0 is out
      }
    }
    if constexpr (RWAVES == 2) __syncthreads();
    swapped = true;
    exchanges++;
    sent = __builtin_readcyclecounter();
    if (wave == RW) {
      double more[2] = {INFINITY, INFINITY};      // of the second wave, for the second best
      if constexpr (RWAVES == 2) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const double ov = s_half[h][0], o2 = s_half[h][1];
          const int oi = s_hrow[h];
          const bool t = oi >= 0 && (br[h] < 0 || ov < bv[h]);      // (equal values: the lower row, which is here)
          more[h] = t ? lesser(br[h] < 0 ? INFINITY : bv[h], o2) : oi >= 0 ? ov : INFINITY;
          bv[h] = t ? ov : bv[h]; br[h] = t ? oi : br[h]; bs[h] = t ? s_hslot[h] : bs[h];
        }
      }
      uint64_t* const out = A.sh->word[exchanges & 1][0] + wg;
      const uint64_t tag = (uint64_t)(uint32_t)(run * 256 + exchanges) << 32;
      const int h = lane >= WORDS, k = lane - h * WORDS;
      if constexpr (!GIVEN) {
        __builtin_amdgcn_s_waitcnt(0);      // the columns of C0 before the record that lets others read them
        asm volatile("" ::: "memory");
        const double best = h ? bv[1] : bv[0];
        const int r = h ? br[1] : br[0], sl = h ? bs[1] : bs[0];
        const uint32_t id = r < 0 ? 0u : (1u << 30) | (sl == PEND ? 1u << 29 : (uint32_t)(sl + 1) << 16) | (uint32_t)r;
        const uint32_t x = k == 0 ? (uint32_t)__double2hiint(best) : k == 1 ? (uint32_t)__double2loint(best) : id;
        if (lane < 2 * WORDS && k < 3) show(out + lane * RUN_WGS, tag | x);
      }
      const double m2[2] = {lesser(from_lane(wave_min(b2[0]), 63), more[0]), lesser(from_lane(wave_min(b2[1]), 63), more[1])};
      if constexpr (!GIVEN) {      // for the first workgroup's record of the gaps only
        const double next = h ? m2[1] : m2[0];
        if (lane < 2 * WORDS && k >= 3) show(out + lane * RUN_WGS, tag | (k == 3 ? (uint32_t)__double2hiint(next) : (uint32_t)__double2loint(next)));
      }
      if (lane < 2) {
        s_rec.best[lane] = lane ? bv[1] : bv[0]; s_rec.second[lane] = lane ? m2[1] : m2[0]; s_rec.row[lane] = lane ? br[1] : br[0]; s_rec.slot[lane] = lane ? bs[1] : bs[0];
      }
    }
    if (wave >= RW && wave < RW + RWAVES) __builtin_amdgcn_s_setprio(0);
    // ---- bordering, while the records are on their way
    if (wg == nwg - 1 && tid < 256) {      // K_TT, for the swaps that are a launch each
      const int h = tid >> 7, k = tid & (TM - 1);
      double* KT = args_again()->KT;
      if (k <= tau + 1) {
        const double x = k < tau ? sk[h][k] : s_kk[h + k - tau];
        KT[(tau + h) * TM + k] = x; KT[k * TM + tau + h] = x;
      }
    }
    if (rows_in) {
      // L' = L + a s^T + s a^T + b t^T + t b^T, s = (y11 a + y12 b) / 2 - u1, t = (y22 b + y12 a) / 2 - u2
      const double e11 = 0.5 * y11, e12 = 0.5 * y12, e22 = 0.5 * y22;
#pragma unroll
      for (int v = 0; v < 4; v++) {
        if (32 * v < th) {
          const int c = 32 * v + 2 * l;
          const d2 a = *reinterpret_cast<const d2*>(&sa[0][c]), b = *reinterpret_cast<const d2*>(&sa[1][c]);
          const d2 s = e11 * a + e12 * b - *reinterpret_cast<const d2*>(&sa[2][c]), t = e22 * b + e12 * a - *reinterpret_cast<const d2*>(&sa[3][c]);
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const int r = 4 * rq + i;
            const double ar = sa[0][r], br = sa[1][r], sr = e11 * ar + e12 * br - sa[2][r], tr = e22 * br + e12 * ar - sa[3][r];
            mv[i][v] += (ar * Dg) * a + (br * Dj) * b;
            lv[i][v] += ar * s + sr * a + br * t + tr * b;
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; v++) {
      if (32 * v < th) {
        const bool here = 32 * v + 2 * l == tau;
#pragma unroll
        for (int i = 0; i < R; i++) {
          const int k = R * rq + i;
          const d2 n = d2{s_new[0][k], s_new[1][k]};
          const f2 f = f2{s_c[0][k], s_c[1][k]};
          if (v < GV) gb[i][v] = here ? n : gb[i][v]; else if (here) s_gb[i * RT + tid] = n;
          if constexpr (C_LDS) { if (here) s_c0[(i * 4 + v) * RT + tid] = f; } else c4[i][v] = here ? f : c4[i][v];
        }
      }
    }
    tau += 2;
    if constexpr (GIVEN) __syncthreads();      // (between swaps that are picked the barrier of the pick does this)
  }

  // ---- does the run count?
  __syncthreads();      // the last swap's rows
  if constexpr (!GIVEN) {
    if (s_late) stalled = true;
    // without patience (tests) the last workgroup gives up for certain, whether or not it had to wait
    if (A.patience == 0 && swapped) { waited = true; stalled |= wg == nwg - 1; }
  }
  bool counts = !stalled;
  if constexpr (!GIVEN) {
    if (waited) {      // the same in every workgroup
      if (tid == 0) {
        int32_t expect = 0;
        const int32_t want = stalled ? 2 : 1;
        if (!stalled) {
          const int32_t n = __hip_atomic_fetch_add(&A.sh->arrived[run], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (n == nwg - 1) __hip_atomic_compare_exchange_strong(&A.sh->verdict[run], &expect, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
          while (seen(&A.sh->verdict[run]) == 0 && __builtin_amdgcn_s_memrealtime() - t0 < A.patience) __builtin_amdgcn_s_sleep(1);
        }
        expect = 0;      // stalled, or nobody has decided in time: it does not
        __hip_atomic_compare_exchange_strong(&A.sh->verdict[run], &expect, 2, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_flag = seen(&A.sh->verdict[run]);
      }
      __syncthreads();
      counts = s_flag == 1;
    }
  }
  RunArgsPtr E = args_again();
  {
  OSSCAR_RUN_THREAD;
  if (!counts) {      // the state as it was
    if (wg == 0 && tid == 0) { SearchCtrl c = *E->cin; c.stalled = 1; *E->cout = c; }
    if (tid == 0) E->rec2[wg] = E->rec[wg];
    const int tw = min(TM, (tau_start + 31) & ~31);
    for (int u = wg; u < 16; u += nwg) {      // (a loop of its own: beside the results it sent 40 of their registers to memory)
      const int r = 4 * rq + u / 4, c = 32 * (u % 4) + 2 * l;
      if (r < tw && c < tw) {
        *reinterpret_cast<d2*>(E->Minv2 + r * TM + c) = *reinterpret_cast<const d2*>(E->Minv + r * TM + c);
        *reinterpret_cast<d2*>(E->LL2 + r * TM + c) = *reinterpret_cast<const d2*>(E->LL + r * TM + c);
      }
    }
    return;
  }
  const int tw = min(TM, (tau + 31) & ~31);
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int r = 4 * rq + i, c = 32 * v + 2 * l;
      if ((i * 4 + v) % nwg == wg && r < tw && c < tw) {
        *reinterpret_cast<d2*>(E->Minv2 + r * TM + c) = mv[i][v]; *reinterpret_cast<d2*>(E->LL2 + r * TM + c) = lv[i][v];
      }
    }
  if (tid == 0) E->rec2[wg] = s_rec;
  if (swapped && has_row) { E->rho[row] = s_rho[lrow]; E->diag[row] = s_diag[lrow]; E->score[row] = s_score[lrow]; E->kept[row] = s_kept[lrow]; E->pos[row] = s_pos[lrow]; }
  if (wg == 0) {
    if (tid >= tau_start && tid < tau) { E->Tidx[tid] = s_T[tid]; E->Jsg[tid] = (float)s_sign[tid]; E->tslot[tid] = s_slot[tid]; }
    if (tid == 0) {
      SearchCtrl* o = E->cout;
      o->done = done; o->iters = iters; o->accepted = E->cin->accepted + accepted; o->notpd = notpd ? 1 : 0; o->g_out = g_out; o->g_in = g_in;
      o->pause = pause; o->tau = tau; o->tau_inc = 0; o->misses = E->cin->misses; o->obj = s_obj[iters & 1]; o->rel_tol = E->cin->rel_tol;
      o->delta = s_run.delta; o->gap_rem = s_run.gap_rem; o->gap_add = s_run.gap_add; o->stalled = E->cin->stalled; o->spare = E->cin->spare; o->taken = E->cin->taken;
    }
  }
  }
}
#undef OSSCAR_RUN_THREAD

#define OSSCAR_RUN_KERNEL(GIVEN)                                                                               \
  (rows == 32 ? (const void*)swap_run_kernel<32, GIVEN> : rows == 64 ? (const void*)swap_run_kernel<64, GIVEN> \
                                                                     : (const void*)swap_run_kernel<128, GIVEN>)
bool swap_run_fits(int64_t d1) {
  const int rows = swap_rows_per_wg((int)d1), nwg = swap_record_count(d1);
  if (nwg > RUN_WGS) return false;
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, OSSCAR_RUN_KERNEL(false), RT, 0) != hipSuccess)
    return false;
  return (int64_t)cus * per >= nwg;
}

hipError_t launch_swap_run(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, SearchCtrl* next, int always, int limit, int run, uint32_t patience,
                           hipStream_t s, const SwapList& l) {
  if (l.n < 0 || l.n > 64 || (l.n > 0 && (!l.out || !l.in)) || run < 0 || run >= RUN_MOST) return hipErrorInvalidValue;
  const int rows = swap_rows_per_wg(d.d1), nwg = swap_record_count(d.d1);
  if (l.n == 0 && nwg > RUN_WGS) return hipErrorInvalidValue;
  RunArgs a{};
  a.N0 = t.N; a.GbT = L.GbT; a.K = L.K; a.C0R = L.C0R; a.sh = reinterpret_cast<RunShared*>(L.run_shared);
  a.d1 = d.d1; a.nwg = nwg; a.limit = limit; a.run = run; a.list_n = l.n; a.always = always; a.patience = patience;
  a.trace_out = t.trace_out; a.trace_in = t.trace_in; a.trace_gap = t.trace_gap; a.trace_obj = t.trace_obj;
  a.cin = t.ctrl; a.cout = next; a.kept = t.kept; a.pos = L.pos; a.Tidx = L.Tidx; a.tslot = L.tslot; a.cslot = L.cslot; a.Jsg = L.Jsg;
  a.rho = t.gram; a.diag = t.dblk; a.score = t.score; a.Minv = L.Minv; a.Minv2 = L.Minv2; a.KT = L.KT; a.LL = L.LL; a.LL2 = L.LL2; a.rec = L.rec; a.rec2 = L.rec2;
  a.list_g = l.out; a.list_j = l.in; a.list_step = l.step;
  void* args[] = {&a};
  return hipLaunchKernel(l.n > 0 ? OSSCAR_RUN_KERNEL(true) : OSSCAR_RUN_KERNEL(false), dim3(nwg), dim3(RT), args, 0, s);
}

}  // namespace osscar
