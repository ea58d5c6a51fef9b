// Quadratic-form construction (Section 3, dense-layer paragraph): H = X^T X accumulated over chunks of
// calibration rows, then the ridge, G = H W and c0.
//
// gram_pack_kernel + gram_packed_kernel: SYRK-style product on the lower-triangle tiles of H with
//   v_mfma_f32_32x32x16_bf16.  Both MFMA operands are column panels of the same row-major chunk Xc (rows =
//   tokens), so every lane needs 8 consecutive TOKENS of one column in a register quad: the chunk is first
//   rewritten once into that order (8 x 8 register transposes, HBM-bound, a few percent of the product's
//   time), and the product kernel then only copies contiguous blocks into LDS and issues MFMAs.
//   Tile order: the host lays the tiles out so that the workgroups that run together on one XCD (block
//   index modulo 8) form 4 x 8 blocks of tiles sharing their 12 column panels in that XCD's L2.
#include "internal.h"
#include <cstdlib>
#include <type_traits>
#include <vector>

namespace osscar {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int GBK = 64;            // tokens per LDS stage

// Tile order: the tiles in RB x CB blocks, one block after the other, and the whole sequence cut into eight equal parts, one per
// XCD (block index modulo 8 selects the XCD); padded with (-1, -1) to equal length.  The tiles that an XCD works on at a time
// share their panels, and all eight have equal work at every size: with whole strips of 4 tile rows dealt to the XCDs, 2048
// columns kept four XCDs busy, and 4096 columns gave one of them twice the average.
template <typename Keep>
static void deal_tiles(int R, int C, int RB, int CB, Keep keep, std::vector<int2>& out) {
  std::vector<int2> seq;
  for (int r0 = 0; r0 < R; r0 += RB)
    for (int c0 = 0; c0 < C; c0 += CB)
      for (int r = r0; r < std::min(R, r0 + RB); r++)
        for (int c = c0; c < std::min(C, c0 + CB); c++)
          if (keep(r, c)) seq.push_back(int2{r, c});
  const size_t per = (seq.size() + 7) / 8;
  out.assign(per * 8, int2{-1, -1});
  for (size_t i = 0; i < seq.size(); i++) out[(i % per) * 8 + i / per] = seq[i];
}
static void build_tile_list(int tiles, std::vector<int2>& out) {
  deal_tiles(tiles, tiles, 4, 8, [](int r, int c) { return c <= r; }, out);
}

// ------------------------------------------------------------------------------------------------
// gram_pack_kernel rewrites a chunk of X once into the operand format of the MFMA: for every panel (64 columns; always an
// even number of panels) and every stage (64 tokens) one contiguous 8 KB block of 16-byte packets, packet (kg, c) = the 8
// tokens kg*8..kg*8+7 of column c, at slot kg*64 + c.  Tokens past the chunk and columns past d1 are zero.  The stages of a
// panel follow one another: with the panels of a stage side by side every stage of a workgroup lay on other pages (3.7 MB
// on for 28672 columns), and the wide kernel below took 14.7 instead of 13.6 ms for 16384 rows.
// gram_packed_kernel then copies whole blocks global -> LDS (linear, no transposes or masks in the hot loop) and
// reads MFMA operands as single ds_read_b128: 16 neighbouring lanes read 16 neighbouring packets.
// Accuracy: the MFMA accumulators are added (v_add_f32, round to nearest) to a second float32 register set every
// `window` stages and restarted from zero, so the accumulation inside the matrix core never spans more than
// window*64 tokens; the second set is added to the float64 H at the end of every range of the contraction.  (The wide kernel's
// second set is float64.)
// ------------------------------------------------------------------------------------------------
constexpr int PK_SLOTS = 8 * 64;    // packets per (panel, stage)
// first packet of the 8 x 8 block (kg, columns 8 cg ..) of a pair of panels in a stage; pstages: stages that a panel has room for
__device__ __forceinline__ int64_t pack_slot(int pair, int pstages, int stage, int kg, int cg) {
  return ((int64_t)(pair * 2 + (cg >> 3)) * pstages + stage) * PK_SLOTS + kg * 64 + (cg & 7) * 8;
}

__global__ __launch_bounds__(256) void gram_pack_kernel(const uint16_t* __restrict__ X, int64_t n_c, int64_t ldx, int d1,
                                                         int npanels, uint4* __restrict__ Xp, int pstages, int stage0) {
  const int tid = threadIdx.x;
  const int panel = blockIdx.x * 2 + (tid >> 7);
  if (panel >= npanels) return;
  const int kg = (tid & 127) >> 4, cg = tid & 15;
  const int col = panel * 128 + cg * 8;
  const bool live = col < d1;
  const int64_t row0 = (int64_t)blockIdx.y * GBK + kg * 8;
  const uint16_t* src = X + (live ? col : 0);
  uint4 st[8];
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int64_t row = row0 + r;
    const int64_t rowc = row < n_c ? row : n_c - 1;
    st[r] = *reinterpret_cast<const uint4*>(src + rowc * ldx);
  }
#pragma unroll
  for (int r = 0; r < 8; r++)
    if (!live || row0 + r >= n_c) st[r] = uint4{0u, 0u, 0u, 0u};
  uint4* out = Xp + pack_slot(panel, pstages, stage0 + blockIdx.y, kg, cg);
#define OSSCAR_PACK_LO(F) uint4{(st[0].F & 0xFFFFu) | (st[1].F << 16), (st[2].F & 0xFFFFu) | (st[3].F << 16), \
                                (st[4].F & 0xFFFFu) | (st[5].F << 16), (st[6].F & 0xFFFFu) | (st[7].F << 16)}
#define OSSCAR_PACK_HI(F) uint4{(st[0].F >> 16) | (st[1].F & 0xFFFF0000u), (st[2].F >> 16) | (st[3].F & 0xFFFF0000u), \
                                (st[4].F >> 16) | (st[5].F & 0xFFFF0000u), (st[6].F >> 16) | (st[7].F & 0xFFFF0000u)}
  out[0] = OSSCAR_PACK_LO(x); out[1] = OSSCAR_PACK_HI(x);
  out[2] = OSSCAR_PACK_LO(y); out[3] = OSSCAR_PACK_HI(y);
  out[4] = OSSCAR_PACK_LO(z); out[5] = OSSCAR_PACK_HI(z);
  out[6] = OSSCAR_PACK_LO(w); out[7] = OSSCAR_PACK_HI(w);
#undef OSSCAR_PACK_LO
#undef OSSCAR_PACK_HI
}

// The same repacking for a convolutional layer: the 8 x 8 blocks are gathered from the feature map, patch by patch.
__global__ __launch_bounds__(256) void gram_pack_conv_kernel(const uint16_t* __restrict__ F, ConvSpec cs, int64_t r0, int64_t n_c,
                                                              int d1, int npanels, uint4* __restrict__ Xp, int pstages, int stage0) {
  const int tid = threadIdx.x;
  const int panel = blockIdx.x * 2 + (tid >> 7);
  if (panel >= npanels) return;
  const int kg = (tid & 127) >> 4, cg = tid & 15;
  const int col0 = panel * 128 + cg * 8;
  const int64_t row0 = (int64_t)blockIdx.y * GBK + kg * 8;
  const int kk = cs.kh * cs.kw;
  uint32_t v[8][4];                       // v[j][r/2]: rows r, r+1 of column j
#pragma unroll
  for (int j = 0; j < 8; j++)
#pragma unroll
    for (int h = 0; h < 4; h++) v[j][h] = 0u;
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int64_t row = row0 + r;
    if (row >= n_c) continue;
    const int64_t pr = r0 + row;
    const int ox = (int)(pr % cs.Wout), oy = (int)((pr / cs.Wout) % cs.Hout), b = (int)(pr / ((int64_t)cs.Wout * cs.Hout));
#pragma unroll
    for (int j = 0; j < 8; j++) {
      const int col = col0 + j;
      if (col >= d1) continue;
      const int c = col / kk, dy = (col % kk) / cs.kw, dx = col % cs.kw;
      const int y = oy * cs.stride + dy - cs.pad, x = ox * cs.stride + dx - cs.pad;
      if (y < 0 || y >= cs.Hin || x < 0 || x >= cs.Win) continue;
      const uint32_t e = F[(((int64_t)b * cs.C + c) * cs.Hin + y) * cs.Win + x];
      v[j][r >> 1] |= (r & 1) ? (e << 16) : e;
    }
  }
  uint4* out = Xp + pack_slot(panel, pstages, stage0 + blockIdx.y, kg, cg);
#pragma unroll
  for (int j = 0; j < 8; j++) out[j] = uint4{v[j][0], v[j][1], v[j][2], v[j][3]};
}

// H64 += acc + acc2 for a wave's RT x CT MFMA tiles at (row0, col0); symmetric: on and below the diagonal only.  C layout of the
// 32 x 32 MFMA: register r = rr*4 + r3 holds row rr*8 + (lane/32)*4 + r3, column lane%32.  A workgroup is the only one that
// touches its tile in a launch, so these are plain loads and stores, a batch of 4 CT loads ahead of the batch that is stored
// (or, atomics, additions that the few workgroups of a small launch do not wait for; or, fresh, stores of a part's sums by themselves):
// with atomics throughout 8192 columns, 2048 rows took 0.305 ms, 0.251 so, 0.19 without reading H64.
template <int RT, int CT, typename A2>
__device__ __forceinline__ void add_tile(const f16v (&acc)[RT][CT], const A2 (&acc2)[RT][CT], double* __restrict__ H64, int ldo, int row0,
                                         int col0, int rows_out, int cols_out, int symmetric, int lane, int atomics = 0, int fresh = 0) {
  // opaque: keeps the compiler from computing all the addresses and conditions ahead of the main loop
  int ldv = ldo;
  asm volatile("" : "+s"(ldv), "+v"(lane));
  const int rbase = row0 + (lane >> 5) * 4, cbase = col0 + (lane & 31);
  double* hbase = H64 + (int64_t)rbase * ldv + cbase;
  double old[2][4][CT];
  auto inside = [&](int ro, int b) {
    const int row = rbase + ro, col = cbase + b * 32;
    return row < rows_out && col < cols_out && (!symmetric || col <= row);
  };
  if (atomics) {
#pragma unroll
    for (int batch = 0; batch < RT * 4; batch++)
#pragma unroll
      for (int r3 = 0; r3 < 4; r3++)
#pragma unroll
        for (int b = 0; b < CT; b++) {
          const int a = batch >> 2, r = (batch & 3) * 4 + r3, ro = a * 32 + (batch & 3) * 8 + r3;
          if (inside(ro, b)) unsafeAtomicAdd(hbase + (int64_t)ro * ldv + b * 32, (double)acc[a][b][r] + (double)acc2[a][b][r]);
        }
    return;
  }
  if (fresh) {      // the whole tile: its buffer holds what lies outside the result, too
#pragma unroll
    for (int a = 0; a < RT; a++)
#pragma unroll
      for (int r = 0; r < 16; r++)
#pragma unroll
        for (int b = 0; b < CT; b++) hbase[(int64_t)(a * 32 + (r >> 2) * 8 + (r & 3)) * ldv + b * 32] = (double)acc[a][b][r] + (double)acc2[a][b][r];
    return;
  }
  auto load = [&](int batch) {
#pragma unroll
    for (int r3 = 0; r3 < 4; r3++)
#pragma unroll
      for (int b = 0; b < CT; b++) {
        const int ro = (batch >> 2) * 32 + (batch & 3) * 8 + r3;
        old[batch & 1][r3][b] = inside(ro, b) ? hbase[(int64_t)ro * ldv + b * 32] : 0.0;
      }
  };
  load(0);
#pragma unroll
  for (int batch = 0; batch < RT * 4; batch++) {
    if (batch + 1 < RT * 4) load(batch + 1);
#pragma unroll
    for (int r3 = 0; r3 < 4; r3++)
#pragma unroll
      for (int b = 0; b < CT; b++) {
        const int a = batch >> 2, r = (batch & 3) * 4 + r3, ro = a * 32 + (batch & 3) * 8 + r3;
        if (inside(ro, b)) hbase[(int64_t)ro * ldv + b * 32] = old[batch & 1][r3][b] + ((double)acc[a][b][r] + (double)acc2[a][b][r]);
      }
    asm volatile("" ::: "memory");
  }
}

// Out (+)= A^T B for packed operands Ap (rows of the result) and Bp (columns of the result); symmetric: Ap == Bp and only
// tiles on or below the diagonal are listed, the diagonal ones loading one operand.  blockIdx.y: the part of the contraction;
// part y is added to copy y of Out (copy_stride doubles apart), so that parts that run side by side never meet.  Sums inside
// the matrix core restart every `window` stages, and every `range` stages (a part is a whole number of ranges) the sums go to
// float64: float32 never spans more than one range.
__global__ __launch_bounds__(256, 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void gram_packed_kernel(
    const uint4* __restrict__ Ap, const uint4* __restrict__ Bp, int pstages, int nstages, int rows_out, int cols_out, int ldo,
    double* __restrict__ H64, int64_t copy_stride, const int2* __restrict__ tile_list, int stages_per_split, int window,
    int range, int symmetric, int atomics) {
  constexpr int WT = 2, TS = 128;
  extern __shared__ uint4 lds[];             // [2 buffers][2 operands][2 panels][PK_SLOTS]
  const int2 tile = tile_list[blockIdx.x];
  if (tile.x < 0) return;
  const int tm = tile.x, tn = tile.y;
  const bool diag = symmetric && (tm == tn);
  const int i0 = tm * TS, j0 = tn * TS;
  const int s_begin = (int)blockIdx.y * stages_per_split;
  H64 += (int64_t)blockIdx.y * copy_stride;
  const int s_end = (s_begin + stages_per_split < nstages) ? s_begin + stages_per_split : nstages;
  if (s_begin >= s_end) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  f16v acc[WT][WT], acc2[WT][WT];
  const int64_t pstride = (int64_t)pstages * PK_SLOTS;
  const uint4* ga = Ap + 2 * tm * pstride + tid;
  const uint4* gb = Bp + 2 * tn * pstride + tid;
  uint4 ra0, ra1, ra2, ra3, rb0, rb1, rb2, rb3;
  rb0 = rb1 = rb2 = rb3 = uint4{0u, 0u, 0u, 0u};
#define OSSCAR_GLOAD(st)                                                                         \
  {                                                                                              \
    const uint4* pa_ = ga + (int64_t)(st) * PK_SLOTS;                                            \
    ra0 = pa_[0]; ra1 = pa_[256]; ra2 = pa_[pstride]; ra3 = pa_[pstride + 256];                  \
    if (!diag) {                                                                                 \
      const uint4* pb_ = gb + (int64_t)(st) * PK_SLOTS;                                          \
      rb0 = pb_[0]; rb1 = pb_[256]; rb2 = pb_[pstride]; rb3 = pb_[pstride + 256];                \
    }                                                                                            \
  }
#define OSSCAR_SSTORE(buf)                                                                       \
  {                                                                                              \
    uint4* la_ = lds + ((buf) * 4 + 0) * PK_SLOTS + tid;                                         \
    la_[0] = ra0; la_[256] = ra1; la_[512] = ra2; la_[768] = ra3;                                \
    if (!diag) {                                                                                 \
      uint4* lb_ = lds + ((buf) * 4 + 2) * PK_SLOTS + tid;                                       \
      lb_[0] = rb0; lb_[256] = rb1; lb_[512] = rb2; lb_[768] = rb3;                              \
    }                                                                                            \
  }
  const int oa = wm * PK_SLOTS + (lane & 31), ob = wn * PK_SLOTS + (lane & 31);

  OSSCAR_GLOAD(s_begin);
  OSSCAR_SSTORE(0);
  __syncthreads();
  int buf = 0;
  for (int r_begin = s_begin; r_begin < s_end; r_begin += range) {
#pragma unroll
    for (int a = 0; a < WT; a++)
#pragma unroll
      for (int b = 0; b < WT; b++)
#pragma unroll
        for (int r = 0; r < 16; r++) { acc[a][b][r] = 0.f; acc2[a][b][r] = 0.f; }
    const int r_end = min(r_begin + range, s_end);
    int in_window = 0;
    for (int st = r_begin; st < r_end; st++) {
      const bool more = (st + 1 < s_end);
      if (more) OSSCAR_GLOAD(st + 1);
      const uint4* pa = lds + (buf * 4 + 0) * PK_SLOTS;
      const uint4* pb = diag ? pa : lds + (buf * 4 + 2) * PK_SLOTS;
      __builtin_amdgcn_s_setprio(1);        // the wave that is multiplying goes first; the other wave of the SIMD issues its loads and stores in between
#pragma unroll
      for (int ks = 0; ks < GBK / 16; ks++) {
        const int kgo = (ks * 2 + (lane >> 5)) * 64;
        bf8 fa[WT], fb[WT];
#pragma unroll
        for (int a = 0; a < WT; a++) {
          uint4 v = pa[kgo + oa + a * 32];
          fa[a] = *reinterpret_cast<bf8*>(&v);
        }
#pragma unroll
        for (int b = 0; b < WT; b++) {
          uint4 v = pb[kgo + ob + b * 32];
          fb[b] = *reinterpret_cast<bf8*>(&v);
        }
#pragma unroll
        for (int a = 0; a < WT; a++)
#pragma unroll
          for (int b = 0; b < WT; b++)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
      }
      __builtin_amdgcn_s_setprio(0);
      if (++in_window >= window && st + 1 < r_end) {
        in_window = 0;
#pragma unroll
        for (int a = 0; a < WT; a++)
#pragma unroll
          for (int b = 0; b < WT; b++)
#pragma unroll
            for (int r = 0; r < 16; r++) { acc2[a][b][r] += acc[a][b][r]; acc[a][b][r] = 0.f; }
      }
      if (more) OSSCAR_SSTORE(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
    add_tile<WT, WT>(acc, acc2, H64, ldo, i0 + wm * 64, j0 + wn * 64, rows_out, cols_out, symmetric, lane, atomics);
  }
#undef OSSCAR_GLOAD
#undef OSSCAR_SSTORE
}

// ------------------------------------------------------------------------------------------------
// The same product in 256 x 192 tiles, one workgroup of 8 waves (64 x 96 each) per compute unit.  The 128 x 128 tile moves
// 64 KB through LDS and 32 KB into it for every 64 MFMAs per SIMD and is bound by that path; here it is 160 KB and 56 KB for
// 192.  Stages of 32 tokens go global -> LDS directly into four buffers of 28 KB, so that three stages are in flight behind
// the one that is read; the operands of a half stage are read while the other half multiplies, and one barrier per stage
// says both that the next stage has landed and that this one's buffer is free.  The buffers are separate arrays and the
// steady loop has no condition: with one array, or with conditional requests, the compiler cannot tell which requests
// a read of LDS depends on and waits for all of them.  16384 rows of 28672 columns, evenly distributed values: 21.0 ms
// that way, 13.6 ms as here, 16.0 ms in 128 x 128 tiles; the layer's own activations: 11.5 against 16.3 ms.  Five buffers
// were 1 % faster still, but their loop cannot end an accumulation window at 1024 tokens.  What bounds it: the matrix cores
// are busy 55 % of the cycles, the requests' way into LDS takes most of the rest, and the clock falls to 1.8 GHz under this load.
// CT = 2: the same in 256 x 128 tiles with the second accumulator set in float64 (the registers of a third column of MFMA tiles),
// which takes every window's sums whole: for the rows of many calls in one launch, whose sums went to the float64 result one call at a time.
// ------------------------------------------------------------------------------------------------
constexpr int GW_R = 256, GW_C = 192, GW_A = 1024;      // packets of A in a 32-token stage: 4 panels (of B: CT panels)
#define OSSCAR_GW_WAIT(n_) __builtin_amdgcn_s_waitcnt(((n_) & 15) | (7 << 4) | (15 << 8) | (((n_) >> 4) << 14))      // vmcnt <= n_
#define OSSCAR_GW_BARRIER()                                                                                        \
  {                                                                                                                \
    asm volatile("" ::: "memory");                                                                                 \
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14)); /* lgkmcnt = 0: all reads of the current buffer are done */ \
    __builtin_amdgcn_s_barrier();                                                                                  \
    asm volatile("" ::: "memory");                                                                                 \
  }
typedef double d16v __attribute__((ext_vector_type(16)));
template <int CT>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_waves_per_eu(2, 2))) void gram_wide_kernel(
    const uint4* __restrict__ Ap, int a_panels, const uint4* __restrict__ Bp, int b_panels, int pstages, int nstages, int rows_out,
    int cols_out, int ldo, double* __restrict__ H64, int64_t copy_stride, const int2* __restrict__ tile_list, int per, int window, int range,
    uint64_t ends_lo, uint64_t ends_hi, int symmetric, int whole, int tail_parts, int tail_per, double* __restrict__ tail_out) {
  constexpr int TC = CT * 64, GW_ST = GW_A + CT * 256;
  typedef typename std::conditional<CT == 2, double, float>::type A2;
  typedef typename std::conditional<CT == 2, d16v, f16v>::type A2v;
  __shared__ uint4 lb0[GW_ST], lb1[GW_ST], lb2[GW_ST], lb3[GW_ST];
  // workgroups from `whole` on: a part of a tile each, whose sums go to a tile of tail_out
  const int in_tail = CT == 2 && (int)blockIdx.x >= whole ? (int)blockIdx.x - whole : -1;
  const int2 tile = tile_list[in_tail >= 0 ? whole + in_tail / tail_parts : (int)blockIdx.x];
  if (tile.x < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int py = (int)blockIdx.y;
  H64 += (int64_t)py * copy_stride;
  if (in_tail >= 0) {
    py = in_tail % tail_parts; per = tail_per; range = 2 * tail_per; ldo = TC;
    H64 = tail_out + (int64_t)in_tail * (GW_R * TC) - ((int64_t)tile.x * GW_R * TC + tile.y * TC);
  }
  // stages of 32 tokens from here on (so are window and range); the part of the contraction that this workgroup takes
  const int part = 2 * per * py, nst = min(2 * nstages, part + 2 * per);
  if (part >= nst) return;
#define OSSCAR_GW_LOAD(st_, buf_)                                                                               \
  {                                                                                                             \
    _Pragma("unroll") for (int i = 0; i < NL; i++)                                                              \
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gp[i] + (int64_t)(st_) * 256), \
                                       (__attribute__((address_space(3))) void*)(buf_ + ldst + i * lstep), 16, 0, 0); \
  }
#define OSSCAR_GW_READ(set_, buf_, ks_)                                                                         \
  {                                                                                                             \
    _Pragma("unroll") for (int a = 0; a < 2; a++) { uint4 v = buf_[oa + (ks_) * 2 * GW_R + a * 32]; fa[set_][a] = *reinterpret_cast<bf8*>(&v); } \
    _Pragma("unroll") for (int b = 0; b < CT; b++) { uint4 v = buf_[ob + (ks_) * 2 * TC + b * 32]; fb[set_][b] = *reinterpret_cast<bf8*>(&v); } \
  }
#define OSSCAR_GW_MULT(set_)                                                                                    \
  _Pragma("unroll") for (int a = 0; a < 2; a++) _Pragma("unroll") for (int b = 0; b < CT; b++)                   \
    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set_][a], fb[set_][b], acc[a][b], 0, 0, 0);
#define OSSCAR_GW_STEADY(st_, cur_, nxt_)                                                                       \
  {                                                                                                             \
    OSSCAR_GW_READ(1, cur_, 1);                                                                                 \
    OSSCAR_GW_MULT(0);                                                                                          \
    OSSCAR_GW_WAIT(2 * NL);                                                                                     \
    OSSCAR_GW_BARRIER();                                                                                        \
    OSSCAR_GW_LOAD((st_) + 4, cur_);                                                                            \
    OSSCAR_GW_READ(0, nxt_, 0);                                                                                 \
    OSSCAR_GW_MULT(1);                                                                                          \
  }
#define OSSCAR_GW_TAIL(st_, cur_, nxt_)                                                                         \
  if ((st_) < end) {                                                                                            \
    OSSCAR_GW_READ(1, cur_, 1);                                                                                 \
    OSSCAR_GW_MULT(0);                                                                                          \
    if ((st_) + 1 < end) {                                                                                      \
      OSSCAR_GW_WAIT(0);                                                                                        \
      OSSCAR_GW_BARRIER();                                                                                      \
      if ((st_) + 4 < end) OSSCAR_GW_LOAD((st_) + 4, cur_);                                                     \
      OSSCAR_GW_READ(0, nxt_, 0);                                                                               \
    }                                                                                                           \
    OSSCAR_GW_MULT(1);                                                                                          \
  }
// a window ends every 1024 tokens (window stages) and where the rows of a call end; four stages ending at st_ + 4 have been added
#define OSSCAR_GW_FOLD(st_)                                                                                     \
  {                                                                                                             \
    const int quad_ = (st_) >> 2;                                                                               \
    in_window += 4;                                                                                             \
    if (in_window >= window || (CT == 2 && (((quad_ < 64 ? ends_lo : ends_hi) >> (quad_ & 63)) & 1))) {         \
      in_window = 0;                                                                                            \
      _Pragma("unroll") for (int a = 0; a < 2; a++) _Pragma("unroll") for (int b = 0; b < CT; b++)               \
        _Pragma("unroll") for (int r = 0; r < 16; r++) { acc2[a][b][r] += (A2)acc[a][b][r]; acc[a][b][r] = 0.f; } \
    }                                                                                                           \
  }
  // Two copies of the loops.  Requests of 64 packets.  Waves 0 - 3: the four kg of one panel of A, four requests per stage; waves
  // 4 - 7: one kg of the CT panels of B, CT requests (the count of a wait is a constant).  Panels past the last one are
  // read from the last one (their results are not written).
  auto run = [&](auto nl) {
    constexpr int NL = decltype(nl)::value;
    for (int beg = part; beg < nst; beg += range) {
      int lv = lane;      // opaque: the addresses are formed again in every range instead of being held while a tile is added
      asm volatile("" : "+v"(lv));
      const uint4* gp[NL];
#pragma unroll
      for (int i = 0; i < NL; i++) {
        if (NL == 4) gp[i] = Ap + (int64_t)min(tile.x * 4 + wave, a_panels - 1) * pstages * PK_SLOTS + i * 64 + lv;
        else gp[i] = Bp + (int64_t)min(tile.y * CT + i, b_panels - 1) * pstages * PK_SLOTS + (wave - 4) * 64 + lv;
      }
      const int ldst = NL == 4 ? wave * 64 : GW_A + (wave - 4) * TC, lstep = NL == 4 ? GW_R : 64;
      // in LDS: A as [kg][256 columns], then B as [kg][TC columns]
      const int oa = (lv >> 5) * GW_R + wm * 64 + (lv & 31), ob = GW_A + (lv >> 5) * TC + wn * (TC / 2) + (lv & 31);
      const int end = min(beg + range, nst);
      bf8 fa[2][2], fb[2][CT];
      f16v acc[2][CT];
      A2v acc2[2][CT];
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < CT; b++)
#pragma unroll
          for (int r = 0; r < 16; r++) { acc[a][b][r] = 0.f; acc2[a][b][r] = (A2)0; }
      if (beg > part) OSSCAR_GW_BARRIER();      // the buffers are about to be filled again
      OSSCAR_GW_LOAD(beg, lb0); OSSCAR_GW_LOAD(beg + 1, lb1);      // a whole number of 64-token stages
      if (beg + 2 < end) { OSSCAR_GW_LOAD(beg + 2, lb2); OSSCAR_GW_LOAD(beg + 3, lb3); }
      if (beg + 4 <= end) OSSCAR_GW_WAIT(3 * NL); else OSSCAR_GW_WAIT(0);
      OSSCAR_GW_BARRIER();
      OSSCAR_GW_READ(0, lb0, 0);
      int in_window = 0, st = beg;
      if (beg + 8 <= end) {
        do {
          OSSCAR_GW_STEADY(st, lb0, lb1); OSSCAR_GW_STEADY(st + 1, lb1, lb2);
          OSSCAR_GW_STEADY(st + 2, lb2, lb3); OSSCAR_GW_STEADY(st + 3, lb3, lb0);
          OSSCAR_GW_FOLD(st);
          st += 4;
        } while (st + 8 <= end);
      }
      for (; st < end; st += 4) {
        OSSCAR_GW_TAIL(st, lb0, lb1); OSSCAR_GW_TAIL(st + 1, lb1, lb2); OSSCAR_GW_TAIL(st + 2, lb2, lb3); OSSCAR_GW_TAIL(st + 3, lb3, lb0);
        if (st + 4 < end) OSSCAR_GW_FOLD(st);      // the last window goes to float64 by itself
      }
      add_tile<2, CT>(acc, acc2, H64, ldo, tile.x * GW_R + wm * 64, tile.y * TC + wn * (TC / 2), rows_out, cols_out, symmetric, lane, 0,
                      in_tail >= 0);
    }
  };
  if (wave < 4) run(std::integral_constant<int, 4>{}); else run(std::integral_constant<int, CT>{});
#undef OSSCAR_GW_LOAD
#undef OSSCAR_GW_READ
#undef OSSCAR_GW_MULT
#undef OSSCAR_GW_STEADY
#undef OSSCAR_GW_TAIL
#undef OSSCAR_GW_FOLD
}

// Tiles of the wide kernel (blocks of 1024 x 1536).  symmetric: tiles that hold an element on or below the diagonal.
void wide_tile_list_host(int rows, int cols, bool symmetric, std::vector<int2>& out) {
  deal_tiles((rows + GW_R - 1) / GW_R, (cols + GW_C - 1) / GW_C, 4, 8,
             [&](int r, int c) { return !symmetric || c * GW_C <= std::min(rows, (r + 1) * GW_R) - 1; }, out);
}
// The same for its 256 x 128 tiles (blocks of 1024 x 1024).
void tall_tile_list_host(int rows, int cols, bool symmetric, std::vector<int2>& out) {
  deal_tiles((rows + GW_R - 1) / GW_R, (cols + 127) / 128, 4, 8, [&](int r, int c) { return !symmetric || c * 128 <= std::min(rows, (r + 1) * GW_R) - 1; }, out);
}
size_t wide_tile_entries(int64_t rows, int64_t cols) { return (size_t)((rows + GW_R - 1) / GW_R * ((cols + GW_C - 1) / GW_C) + 8); }

// Rows r0 .. r0 + nr of the patch matrix as float32 (float32 maps and bf16 maps of other than a multiple of eight columns).
// Thread = one column of 16 patches, so that writes run along the rows; bound by writing the rows (115 MB in 0.06 ms).  Idx: type
// of a patch's number, 64 bits wide only if the map has more than 2^31 - 1 patches.
template <typename Idx>
__global__ __launch_bounds__(256) void im2col_rows_kernel(const void* __restrict__ F, int is_bf16, ConvSpec cs, int64_t r0, int64_t nr,
                                                           int d1, float* __restrict__ out) {
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= d1) return;
  const int kk = cs.kh * cs.kw, c = col / kk, dy = (col % kk) / cs.kw - cs.pad, dx = col % cs.kw - cs.pad;
  for (int u = 0; u < 16; u++) {
    const int64_t r = (int64_t)blockIdx.y * 16 + u;
    if (r >= nr) return;
    const Idx pr = (Idx)(r0 + r), line = pr / (Idx)cs.Wout;        // the same for the whole workgroup
    const int ox = (int)(pr % (Idx)cs.Wout), oy = (int)(line % (Idx)cs.Hout), b = (int)(line / (Idx)cs.Hout);
    const int y = oy * cs.stride + dy, x = ox * cs.stride + dx;
    float v = 0.f;
    if (y >= 0 && y < cs.Hin && x >= 0 && x < cs.Win) {
      const int64_t at = (((int64_t)b * cs.C + c) * cs.Hin + y) * cs.Win + x;
      v = is_bf16 ? __uint_as_float(((uint32_t)reinterpret_cast<const uint16_t*>(F)[at]) << 16) : reinterpret_cast<const float*>(F)[at];
    }
    out[r * d1 + col] = v;
  }
}
hipError_t launch_im2col_rows(const void* F, int is_bf16, const ConvSpec& cs, int64_t r0, int64_t nr, int d1, float* out, hipStream_t s) {
  if (nr <= 0) return hipSuccess;
  const dim3 grid((d1 + 255) / 256, (unsigned)((nr + 15) / 16));
  if ((int64_t)cs.Hout * cs.Wout <= INT32_MAX / std::max(cs.B, 1)) hipLaunchKernelGGL(im2col_rows_kernel<uint32_t>, grid, dim3(256), 0, s, F, is_bf16, cs, r0, nr, d1, out);
  else hipLaunchKernelGGL(im2col_rows_kernel<uint64_t>, grid, dim3(256), 0, s, F, is_bf16, cs, r0, nr, d1, out);
  return hipGetLastError();
}

// host-only view of the schedule for tests: fills out[0 .. 2*count) with (row, column) pairs, returns the list length
int gram_tile_schedule(int tiles_per_side, int32_t* out, int capacity) {
  std::vector<int2> t;
  build_tile_list(tiles_per_side, t);
  if (out)
    for (size_t i = 0; i < t.size() && (int)i < capacity; i++) { out[2 * i] = t[i].x; out[2 * i + 1] = t[i].y; }
  return (int)t.size();
}

// How many copies of a float64 result of this many elements and 128 x 128 tiles are kept, so that ranges of the contraction
// can run side by side, each into its own copy: enough for 512 workgroups (two per compute unit), in at most 320 MB.
int packed_copies(int64_t elems, int64_t ntiles) {
  return (int)std::max<int64_t>(1, std::min({(int64_t)16, 512 / std::max<int64_t>(ntiles, 1), ((int64_t)320 << 20) / (8 * elems)}));
}

void gram_tile_list_host(int d1, std::vector<int2>& out) { build_tile_list((d1 + 127) / 128, out); }
void rect_tile_list_host(int d1, int m, std::vector<int2>& out) {
  deal_tiles((d1 + 127) / 128, (m + 127) / 128, 4, 8, [](int, int) { return true; }, out);
}

__global__ void fill_zero_f64_kernel(double* __restrict__ p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0.0;
}

// Out += A^T B over all stages, one launch.  The contraction falls into ranges, as many as bring 2048 tiles together, of at
// least 8 stages: at their ends the sums go to float64, because the error of a float32 sum grows with its length (3000 columns of
// ReLU rows, 16384 of them: rms 1.4e-8 of sqrt(H_ii H_jj), float32's rounding of H included, against 2.6e-8 joined in float32; the
// additions cost 0.05 of 0.33 ms, and 0.01 of 0.052 ms at 2048 columns, 2048 rows).
// From GW_MIN_TILES wide tiles (half of the compute units) and GW_MIN_STAGES stages on: the wide kernel, if its windows of 1024
// tokens end with the ranges (8192 columns, 2048 rows: 0.21 ms, 0.35 in 128 x 128 tiles; 4096 columns, 16384 rows: 0.36 and 0.69).
// Else 128 x 128 tiles, two workgroups per compute unit; when there are too few of them for the chip, the ranges are dealt to
// up to acc.copies workgroups per tile, each adding to its own copy of Out; the caller adds the copies up in order (2048
// columns, 2048 rows: 0.052 ms, 0.084 as four launches one after the other).
// Rows of several calls (launch_gram_queue): 256 x 128 tiles with float64 windows, Out touched once.
// Either way an element of a copy receives its additions from one thread, in order, so the result does not depend on scheduling.
constexpr size_t GW_MIN_TILES = 128;
constexpr int GW_MIN_STAGES = 32, GW_MIN_PART = 16, LONG_STAGES = 72;
// A launch of the 128 x 128 kernel with fewer workgroups than this adds with atomics, which nobody waits for: 64 columns, 64 rows 7.7 us
// against 11.3 with loads and stores, 1000 columns, 512 rows (36 workgroups) 13.7 and 18.7; 1000 columns, 2048 rows (144) 27.9 both;
// 2048 columns, 2048 rows (272) 67.6 and 51.3.  Either way one thread adds to an element, in order.
constexpr int64_t PLAIN_FROM = 128;
// stages of a range of the 128 x 128 kernel
static int packed_range(int nstages, int ntiles) {
  const int ranges = ntiles < 1024 ? std::min(nstages, (2048 + ntiles - 1) / ntiles) : 1;
  return std::max((nstages + ranges - 1) / ranges, std::min(nstages, 8));
}
// copies of a result that no earlier launch has used
static void clear_copies(const PackedAcc& acc, int parts, int64_t elems, hipStream_t s) {
  if (!acc.cleared || *acc.cleared >= parts) return;
  hipLaunchKernelGGL(fill_zero_f64_kernel, dim3(2048), dim3(256), 0, s, acc.out + *acc.cleared * elems, (parts - *acc.cleared) * elems);
  *acc.cleared = parts;
}
static bool takes_wide(const PackedTiles& t, int nstages, int ntiles, int window) {
  const int range = packed_range(nstages, ntiles);
  return t.wide && t.wide_entries >= GW_MIN_TILES && nstages >= GW_MIN_STAGES && (range >= nstages || range % window == 0);
}
static hipError_t launch_packed(const uint4* Ap, const uint4* Bp, int pstages, int nstages, int rows_out, int cols_out, const PackedAcc& acc,
                                const PackedTiles& t, int ntiles, int window, int symmetric, hipStream_t s) {
  const int range = packed_range(nstages, ntiles), ranges = (nstages + range - 1) / range;
  const int64_t elems = (int64_t)rows_out * cols_out;
  if (takes_wide(t, nstages, ntiles, window)) {
    hipLaunchKernelGGL(gram_wide_kernel<3>, dim3((unsigned)t.wide_entries), dim3(512), 0, s, Ap, (rows_out + 127) / 128 * 2, Bp,
                       (cols_out + 127) / 128 * 2, pstages, nstages, rows_out, cols_out, cols_out, acc.out, elems, t.wide, nstages, 2 * window,
                       2 * range, 0ull, 0ull, symmetric, 0, 1, 0, (double*)nullptr);
    return hipGetLastError();
  }
  const int per = (ranges + acc.copies - 1) / acc.copies * range, parts = (nstages + per - 1) / per;
  clear_copies(acc, parts, elems, s);
  hipLaunchKernelGGL(gram_packed_kernel, dim3((unsigned)t.entries, (unsigned)parts), dim3(256), (size_t)2 * 4 * PK_SLOTS * 16, s, Ap, Bp, pstages,
                     nstages, rows_out, cols_out, cols_out, acc.out, elems, t.list, per, window, range, symmetric,
                     (int64_t)ntiles * parts < PLAIN_FROM);
  return hipGetLastError();
}
// Parts that the contraction of a queued product is cut into, each with its copy of the result: one workgroup per compute unit, and
// at least GW_MIN_PART stages each (512 to 3000 columns, two to four calls of 64 to 6000 rows: 8, 16 and 32 within the 5 % by which runs
// differ, with 4 calls of 256 to 512 rows 3 - 8 % slower; with 32, 512 columns do not fill the chip and their rows do not wait)
static int queue_parts(int nstages, const PackedTiles& t, int copies) {
  return std::max(1, std::min({copies, nstages / GW_MIN_PART, (int)((256 + t.tall_entries - 1) / t.tall_entries)}));
}
// half of the compute units have a workgroup of a queued product
static bool queue_fills(int nstages, const PackedTiles& t, int copies) {
  return t.tall && t.tall_entries > 0 && t.tall_entries * queue_parts(nstages, t, copies) >= GW_MIN_TILES;
}
// Out += the parts of the tiles that were cut, in order: 16 rows of a tile per workgroup, a column of eight per thread, so that a row is read as a
// whole.  Bound by reading the parts (64 MB at most).
__global__ __launch_bounds__(256) void gram_tail_kernel(const double* __restrict__ parts_in, int parts, const int2* __restrict__ tiles, int rows_out, int cols_out,
                                                         double* __restrict__ out, int symmetric) {
  const int2 tile = tiles[blockIdx.x];
  if (tile.x < 0) return;
  const int c = threadIdx.x & 127, r0 = blockIdx.y * 16 + (threadIdx.x >> 7) * 8;
  const int col = tile.y * 128 + c;
  const double* in = parts_in + (int64_t)blockIdx.x * parts * (GW_R * 128) + r0 * 128 + c;
  double v[8];
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int row = tile.x * GW_R + r0 + r;
    v[r] = row < rows_out && col < cols_out && (!symmetric || col <= row) ? out[(int64_t)row * cols_out + col] : 0.0;
  }
  for (int p = 0; p < parts; p++)
#pragma unroll
    for (int r = 0; r < 8; r++) v[r] += in[(int64_t)p * (GW_R * 128) + r * 128];
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int row = tile.x * GW_R + r0 + r;
    if (row < rows_out && col < cols_out && (!symmetric || col <= row)) out[(int64_t)row * cols_out + col] = v[r];
  }
}
static hipError_t launch_queued(const PackedGram& g, const uint4* Ap, const uint4* Bp, int window, int rows_out, int cols_out, const PackedAcc& acc,
                                const PackedTiles& t, int symmetric, hipStream_t s) {
  const PackQueue& q = *g.q;
  const int64_t elems = (int64_t)rows_out * cols_out;
  const int most = queue_parts(q.stages, t, acc.copies), per = ((q.stages + most - 1) / most + 1) / 2 * 2, parts = (q.stages + per - 1) / per;
  clear_copies(acc, parts, elems, s);
  // Tiles that do not fill a last round of the 256 compute units (one workgroup each) are cut along the rows, as many parts of at least
  // GW_MIN_PART stages as fill one, and the parts' sums added up by a second launch.  16384 rows in calls of 2048, repacking included: 4096
  // columns (272 tiles) 487 us whole, 361 so; 8192 (1056) 1330 and 1240; 9216 (1332, cut in four) 1690 and 1580.
  const int left = (int)(t.tall_entries % 256), rounds = (int)(t.tall_entries / 256);
  int cut = 1;
  if (parts == 1 && rounds > 0 && left > 0)
    cut = std::min({256 / left, q.stages / GW_MIN_PART, (int)std::min<size_t>(256, g.spare_bytes / ((size_t)left * GW_R * 128 * 8))});
  int tail_per = q.stages;
  if (cut > 1) { tail_per = ((q.stages + cut - 1) / cut + 1) / 2 * 2; cut = (q.stages + tail_per - 1) / tail_per; }
  const int whole = cut > 1 ? rounds * 256 : (int)t.tall_entries;
  hipLaunchKernelGGL(gram_wide_kernel<2>, dim3((unsigned)(cut > 1 ? whole + left * cut : whole), (unsigned)parts), dim3(512), 0, s, Ap,
                     (rows_out + 127) / 128 * 2, Bp, (cols_out + 127) / 128 * 2, g.pack_stages, q.stages, rows_out, cols_out, cols_out, acc.out, elems, t.tall,
                     per, 2 * window, 2 * per, q.ends[0], q.ends[1], symmetric, whole, std::max(cut, 1), tail_per, g.spare);
  if (cut > 1)
    hipLaunchKernelGGL(gram_tail_kernel, dim3((unsigned)left, GW_R / 16), dim3(256), 0, s, g.spare, cut, t.tall + whole, rows_out, cols_out, acc.out, symmetric);
  return hipGetLastError();
}

// Rows of calls that are shorter than pack_x (and pack_y) wait there until it is full: a launch per call of 2048 rows reads and writes all of
// the float64 result for them.  Every call's rows begin a window of their own and the windows are no longer than the call by itself
// would make them, so no float32 sum is longer than in a launch per call.  16384 rows in calls of 2048: 8192 columns 1.23 ms (8 launches of
// 0.20 before), 2048 columns 0.093 ms (8 of 0.043); the error of H is the same (rms 1.29e-8 and 9.2e-9 of sqrt(H_ii H_jj) either way).
hipError_t launch_gram_queue(const PackedGram& g, hipStream_t s) {
  PackQueue& q = *g.q;
  if (q.stages == 0) return hipSuccess;
  const int npairs = (g.d1 + 127) / 128, npairs_y = g.pack_y ? (g.m + 127) / 128 : 0;
  const uint4 *Xp = reinterpret_cast<const uint4*>(g.pack_x), *Yp = reinterpret_cast<const uint4*>(g.pack_y);
  // Rows that wait when the layer ends may fill fewer workgroups.  Calls of up to GW_MIN_PART stages are still multiplied together, longer
  // ones each in a launch of its own, cut into as many ranges as it can be (512 columns, two calls of 6000 rows, whole quadratic form:
  // 0.40 ms in one launch of eight workgroups, 0.29 so; 1280 columns, three calls of 1024 rows: 0.35 ms together, 0.38 apart).
  auto ends = [&](int stage) { const int pair = stage / 2 - 1; return ((q.ends[pair >> 6] >> (pair & 63)) & 1) != 0; };      // stage: even, above 0
  auto product = [&](const uint4* Bp, int window, int cols, const PackedAcc& acc, const PackedTiles& t, int ntiles, int symmetric) -> hipError_t {
    const bool together = q.calls > 1 && (q.stages <= q.calls * GW_MIN_PART || queue_fills(q.stages, t, acc.copies));
    for (int st = 0, end; st < q.stages; st = end) {
      for (end = together ? q.stages : st + 2; end < q.stages && !ends(end);) end += 2;
      const int n = q.calls > 1 ? end - st : q.last;
      const int64_t at = (int64_t)st * PK_SLOTS;
      const bool timed = symmetric && g.ev && q.ev_used < g.ev_pairs;
      if (timed) hipEventRecord(g.ev[2 * q.ev_used], s);
      const hipError_t e = together ? launch_queued(g, Xp, Bp, window, g.d1, cols, acc, t, symmetric, s)
                                    : launch_packed(Xp + at, Bp + at, g.pack_stages, n, g.d1, cols, acc, t, ntiles, 16, symmetric, s);
      if (e != hipSuccess) return e;
      if (timed) { hipEventRecord(g.ev[2 * q.ev_used + 1], s); q.ev_used++; q.ev_rows += (together || q.calls == 1) ? q.rows : std::min<int64_t>(n * GBK, q.rows); }
    }
    return hipSuccess;
  };
  hipError_t e = product(Xp, q.window, g.d1, g.H64, g.tiles, npairs * (npairs + 1) / 2, 1);
  if (e == hipSuccess && g.pack_y) e = product(Yp, q.window_y, g.m, g.G64, g.tiles_y, npairs * npairs_y, 0);
  q.clear();
  return e;
}
hipError_t launch_gram_packed(const PackedGram& g, const void* Xc, int64_t n_c, int64_t ldx, const void* Yc, int64_t ldy, const ConvSpec* conv,
                              hipStream_t s) {
  PackQueue& q = *g.q;
  if (n_c <= 0) return hipSuccess;
  if (g.pack_stages < 2 || g.pack_stages > 256 || g.pack_stages % 2 || !g.tiles.list || g.tiles.entries == 0) return hipErrorInvalidValue;
  if (Yc && (!g.pack_y || !g.tiles_y.list || g.tiles_y.entries == 0)) return hipErrorInvalidValue;
  const int npairs = (g.d1 + 127) / 128, npairs_y = Yc ? (g.m + 127) / 128 : 0, ntiles = npairs * (npairs + 1) / 2;
  // A call that fills the buffer by itself is multiplied by itself, its last rows included: they are a small part of it, and its H does not
  // depend on the calls around it.  So is one of more than LONG_STAGES where the wide tiles fill four fifths of their rounds of the
  // compute units: from there on the wide kernel's higher rate is more than the pass over the result that waiting would save (whole
  // quadratic form, rows that wait / calls by themselves: 8192 columns, two calls of 4608 rows 2.06 / 2.01 ms, of 8192 rows 2.64 / 2.45, three of
  // 12000 rows 4.34 / 3.78; 28672 columns, three of 12000 41.6 / 38.5, of 4096 20.1 / 20.5; 5120 columns, 287 tiles, two of 8192 rows 1.18 / 1.43).
  const bool whole = n_c >= (int64_t)g.pack_stages * GBK ||
                     (n_c > (int64_t)LONG_STAGES * GBK && g.tiles.wide_entries * 5 >= (g.tiles.wide_entries + 255) / 256 * 256 * 4 &&
                      takes_wide(g.tiles, (int)((n_c + GBK - 1) / GBK), ntiles, 16));
  if (whole) {
    const hipError_t e = launch_gram_queue(g, s);
    if (e != hipSuccess) return e;
  }
  const bool waits = !whole && queue_fills(g.pack_stages, g.tiles, g.H64.copies) && (!Yc || queue_fills(g.pack_stages, g.tiles_y, g.G64.copies));
  for (int64_t r0 = 0; r0 < n_c;) {
    const int64_t nr = std::min<int64_t>((int64_t)(g.pack_stages - q.stages) * GBK, n_c - r0);
    const int nst = (int)((nr + GBK - 1) / GBK), used = (nst + 1) / 2 * 2;      // an even number of stages: the wide kernel's windows
    if (conv)
      hipLaunchKernelGGL(gram_pack_conv_kernel, dim3((npairs + 1) / 2, used), dim3(256), 0, s, reinterpret_cast<const uint16_t*>(Xc),
                         *conv, r0, nr, g.d1, npairs, reinterpret_cast<uint4*>(g.pack_x), g.pack_stages, q.stages);
    else
      hipLaunchKernelGGL(gram_pack_kernel, dim3((npairs + 1) / 2, used), dim3(256), 0, s, reinterpret_cast<const uint16_t*>(Xc) + r0 * ldx, nr, ldx,
                         g.d1, npairs, reinterpret_cast<uint4*>(g.pack_x), g.pack_stages, q.stages);
    if (Yc)
      hipLaunchKernelGGL(gram_pack_kernel, dim3((npairs_y + 1) / 2, used), dim3(256), 0, s, reinterpret_cast<const uint16_t*>(Yc) + r0 * ldy, nr, ldy,
                         g.m, npairs_y, reinterpret_cast<uint4*>(g.pack_y), g.pack_stages, q.stages);
    q.stages += used; q.last = nst; q.rows += nr; q.calls++;
    auto shorten = [&](int& window, int range) { if (range < nst) window = std::min(window, std::max(2, range / 2 * 2)); };
    shorten(q.window, packed_range(nst, ntiles));
    if (Yc) shorten(q.window_y, packed_range(nst, npairs * npairs_y));
    const int pair = q.stages / 2 - 1;
    q.ends[pair >> 6] |= 1ull << (pair & 63);
    r0 += nr;
    if (!waits || q.stages == g.pack_stages) {
      const hipError_t e = launch_gram_queue(g, s);
      if (e != hipSuccess) return e;
    }
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// G = H W on the bf16 matrix cores for bf16 W: H (float32) is split into three bf16 pieces H = H1 + H2 + H3 (each the
// round-to-nearest bf16 of what the previous ones left, so the sum is exact to 2^-25), and H_i^T W = H_i W (H is
// symmetric) runs on the packed kernel above: products of two bf16 numbers are exact in float32, the accumulation is
// restarted every 1024 rows and ends in float64, as for the Gram.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t bf16_rne_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
// piece 0, 1, 2 of the split, packed like gram_pack_kernel packs a bf16 matrix (rows = the contraction index)
__global__ __launch_bounds__(256) void gram_pack_split_kernel(const float* __restrict__ A, int64_t n_c, int64_t lda, int cols,
                                                               int npanels, int piece, uint4* __restrict__ Xp) {
  const int tid = threadIdx.x;
  const int panel = blockIdx.x * 2 + (tid >> 7);
  if (panel >= npanels) return;
  const int kg = (tid & 127) >> 4, cg = tid & 15;
  const int col = panel * 128 + cg * 8;
  const bool live = col < cols;
  const int64_t row0 = (int64_t)blockIdx.y * GBK + kg * 8;
  uint32_t h[8][8];
#pragma unroll
  for (int r = 0; r < 8; r++) {
    const int64_t row = row0 + r;
    float v[8];
    if (live && row < n_c) {
      const float4 a = *reinterpret_cast<const float4*>(A + row * lda + col);
      const float4 b = *reinterpret_cast<const float4*>(A + row * lda + col + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
      for (int j = 0; j < 8; j++) v[j] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 8; j++) {
      float x = v[j];
      uint32_t bits = bf16_rne_bits(x);
      for (int p = 0; p < piece; p++) { x -= __uint_as_float(bits << 16); bits = bf16_rne_bits(x); }
      h[r][j] = bits;
    }
  }
  uint4* out = Xp + pack_slot(panel, gridDim.y, blockIdx.y, kg, cg);
#pragma unroll
  for (int j = 0; j < 8; j++)
    out[j] = uint4{h[0][j] | (h[1][j] << 16), h[2][j] | (h[3][j] << 16), h[4][j] | (h[5][j] << 16), h[6][j] | (h[7][j] << 16)};
}

// G64 (d1 x m, float64, zeroed by the caller) += H W.  H: d1 x d1 float32 (ld = d1, d1 % 8 == 0, 16-byte aligned), W: d1 x m bf16
// (m % 8 == 0, ldw % 8 == 0, 16-byte aligned).  pack_h: pack_rows * 128*ceil(d1/128) * 2 bytes, pack_w likewise for m.
hipError_t launch_hw_split(const float* H, int d1, const void* W, int64_t ldw, int m, double* G64, const PackedTiles& tiles,
                           void* pack_h, void* pack_w, int64_t pack_rows, hipStream_t s) {
  if (pack_rows < GBK || pack_rows % GBK || !tiles.list || tiles.entries == 0) return hipErrorInvalidValue;
  const int npanels = (d1 + 127) / 128, npanels_w = (m + 127) / 128;
  const int window = 16;
  for (int64_t r0 = 0; r0 < d1; r0 += pack_rows) {
    const int64_t nr = std::min<int64_t>(pack_rows, d1 - r0);
    const int nstages = (int)((nr + GBK - 1) / GBK);
    hipLaunchKernelGGL(gram_pack_kernel, dim3((npanels_w + 1) / 2, nstages), dim3(256), 0, s,
                       reinterpret_cast<const uint16_t*>(W) + r0 * ldw, nr, ldw, m, npanels_w, reinterpret_cast<uint4*>(pack_w), nstages, 0);
    for (int piece = 0; piece < 3; piece++) {
      hipLaunchKernelGGL(gram_pack_split_kernel, dim3((npanels + 1) / 2, nstages), dim3(256), 0, s, H + r0 * d1, nr, (int64_t)d1, d1,
                         npanels, piece, reinterpret_cast<uint4*>(pack_h));
      const hipError_t e = launch_packed(reinterpret_cast<const uint4*>(pack_h), reinterpret_cast<const uint4*>(pack_w), nstages, nstages, d1, m,
                                         PackedAcc{G64, 1, nullptr}, tiles, npanels * npanels_w, window, 0, s);
      if (e != hipSuccess) return e;
    }
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// General products of float32 matrices on the bf16 matrix cores: C = beta Cin + alpha A^T B with A (K x M) and B (K x N)
// row-major, the contraction running over their rows.  Each operand is cut into three bf16 pieces (a = a1 + a2 + a3, each the
// round-to-nearest bf16 of what the pieces before it leave: together 24 significand bits), and the six products whose
// weight is at least 2^-16 of the leading one -- a1 b1, a1 b2, a2 b1, a2 b2, a1 b3, a3 b1 -- run on the packed kernel above:
// products of bf16 numbers are exact in float32, sums restart every 1024 rows and end in float64.  What is dropped (a2 b3,
// a3 b2, a3 b3) is below 2^-24 of |a| |b| term by term, the size of the operands' own float32 rounding.
// ------------------------------------------------------------------------------------------------
static int64_t split_kpad(int64_t K) { return (K + GBK - 1) / GBK * GBK; }
size_t split_pack_bytes(int64_t K, int64_t cols) { return (size_t)3 * split_kpad(K) * ((cols + 127) / 128 * 128) * 2; }

hipError_t launch_pack_pieces(const float* A, int64_t lda, int64_t K, int cols, void* pack, hipStream_t s) {
  if (K <= 0 || cols <= 0) return hipSuccess;
  if (cols % 8 || lda % 4 || (reinterpret_cast<uintptr_t>(A) & 15)) return hipErrorInvalidValue;
  const int npanels = (cols + 127) / 128, nstages = (int)(split_kpad(K) / GBK);
  const size_t piece = (size_t)nstages * npanels * 2 * PK_SLOTS;      // uint4 packets per piece
  for (int pc = 0; pc < 3; pc++)
    hipLaunchKernelGGL(gram_pack_split_kernel, dim3((npanels + 1) / 2, nstages), dim3(256), 0, s, A, K, lda, cols, npanels, pc,
                       reinterpret_cast<uint4*>(pack) + pc * piece);
  return hipGetLastError();
}

__global__ void split_epilogue_kernel(const double* __restrict__ acc, int M, int N, const float* __restrict__ Cin, int64_t ldcin,
                                      float* __restrict__ C, int64_t ldc, double alpha, double beta) {
  const int64_t tot = (int64_t)M * N;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = idx / N, j = idx % N;
    double v = alpha * acc[idx];
    if (Cin) v += beta * (double)Cin[i * ldcin + j];
    C[i * ldc + j] = (float)v;
  }
}

// acc (M x N float64, dense) = A^T B from packed pieces; nprod = 6 (full float32 accuracy) or 3 (a1 b1 + a1 b2 + a2 b1: 2^-16)
hipError_t launch_split_product(const void* packA, int M, const void* packB, int N, int64_t K, int nprod, double* acc,
                                const PackedTiles& tiles, int ntiles, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!tiles.list || tiles.entries == 0 || (nprod != 6 && nprod != 3)) return hipErrorInvalidValue;
  const int npa = (M + 127) / 128, npb = (N + 127) / 128, nstages = (int)(split_kpad(K) / GBK);
  const size_t pieceA = (size_t)nstages * npa * 2 * PK_SLOTS, pieceB = (size_t)nstages * npb * 2 * PK_SLOTS;
  hipError_t e = hipMemsetAsync(acc, 0, (size_t)M * N * 8, s);
  if (e != hipSuccess) return e;
  if (K <= 0) return hipSuccess;
  static const int combo[6][2] = {{0, 0}, {0, 1}, {1, 0}, {1, 1}, {0, 2}, {2, 0}};
  for (int c = 0; c < nprod; c++)
    if ((e = launch_packed(reinterpret_cast<const uint4*>(packA) + combo[c][0] * pieceA, reinterpret_cast<const uint4*>(packB) + combo[c][1] * pieceB,
                           nstages, nstages, M, N, PackedAcc{acc, 1, nullptr}, tiles, ntiles, 16, 0, s)) != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_split_epilogue(const double* acc, int M, int N, const float* Cin, int64_t ldcin, float* C, int64_t ldc, double alpha,
                                 double beta, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  hipLaunchKernelGGL(split_epilogue_kernel, dim3(2048), dim3(256), 0, s, acc, M, N, (beta != 0.0) ? Cin : nullptr, ldcin, C, ldc, alpha, beta);
  return hipGetLastError();
}

// sum of squares of a rows x cols matrix (float32 or bf16), added to *acc
__global__ __launch_bounds__(256) void sumsq_kernel(const void* __restrict__ A, int is_bf16, int64_t rows, int64_t cols, int64_t ld,
                                                     double* __restrict__ part) {
  __shared__ double red[4];
  double v = 0;
  const int64_t tot = rows * cols;
  for (int64_t idx = blockIdx.x * 256 + threadIdx.x; idx < tot; idx += (int64_t)gridDim.x * 256) {
    const int64_t r = idx / cols, c = idx % cols;
    const float x = is_bf16 ? __uint_as_float(((uint32_t)reinterpret_cast<const uint16_t*>(A)[r * ld + c]) << 16)
                            : reinterpret_cast<const float*>(A)[r * ld + c];
    v += (double)x * (double)x;
  }
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}
// *acc += the 1024 partial sums, in a fixed order
__global__ __launch_bounds__(1024) void sumsq_add_kernel(const double* __restrict__ part, double* __restrict__ acc);
hipError_t launch_sumsq(const void* A, int is_bf16, int64_t rows, int64_t cols, int64_t ld, double* acc, double* partial, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(sumsq_kernel, dim3(1024), dim3(256), 0, s, A, is_bf16, rows, cols, ld, partial);
  hipLaunchKernelGGL(sumsq_add_kernel, dim3(1), dim3(1024), 0, s, partial, acc);
  return hipGetLastError();
}

// G = float32(G64 + lambda W)
__global__ void finalize_G_kernel(const double* __restrict__ G64, const float* __restrict__ Wf, const double* __restrict__ lambda,
                                  float* __restrict__ G, int64_t n) {
  const double lam = *lambda;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    G[i] = (float)(G64[i] + lam * (double)Wf[i]);
}
hipError_t launch_finalize_G(const double* G64, const float* Wf, const double* lambda_dev, float* G, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(finalize_G_kernel, dim3(2048), dim3(256), 0, s, G64, Wf, lambda_dev, G, n);
  return hipGetLastError();
}

// A (rows x cols) += its copies 1 .. copies - 1 in order; lower: on and below the diagonal only.  Bound by reading the copies
// (32 of 576 columns: 43 MB).
__global__ __launch_bounds__(256) void sum_copies_kernel(double* __restrict__ A, int copies, int rows, int cols, int lower) {
  const int64_t n = (int64_t)rows * cols, i = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (i >= n || (lower && i % cols > i / cols)) return;
  double x = A[i];
#pragma unroll 8
  for (int cp = 1; cp < copies; cp++) x += A[cp * n + i];
  A[i] = x;
}
hipError_t launch_sum_copies(double* A, int copies, int rows, int cols, int lower, hipStream_t s) {
  if (copies <= 1) return hipSuccess;
  hipLaunchKernelGGL(sum_copies_kernel, dim3((unsigned)(((int64_t)rows * cols + 255) / 256)), dim3(256), 0, s, A, copies, rows, cols, lower);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Helpers of the generic (any shape, float32 or bfloat16 input) path and of finalize.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

__global__ void convert_to_f32_kernel(const void* __restrict__ src, int is_bf16, int64_t rows, int64_t cols, int64_t lds_,
                                      float* __restrict__ dst) {
  int64_t n = rows * cols;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int64_t r = i / cols, c = i % cols;
    dst[i] = is_bf16 ? bf16_bits_to_float(reinterpret_cast<const uint16_t*>(src)[r * lds_ + c])
                     : reinterpret_cast<const float*>(src)[r * lds_ + c];
  }
}

hipError_t launch_convert_to_f32(const void* src, int is_bf16, int64_t rows, int64_t cols, int64_t lds_, float* dst,
                                 hipStream_t s) {
  if (rows * cols <= 0) return hipSuccess;
  int blocks = (int)((rows * cols + 1023) / 1024);
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(convert_to_f32_kernel, dim3(blocks), dim3(256), 0, s, src, is_bf16, rows, cols, lds_, dst);
  return hipGetLastError();
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) t += sh[i];
  return t;   // valid in thread 0
}

// H[i][j] = float(H64[max(i,j)][min(i,j)] + (i == j ? lam : 0)).  One workgroup per 64 x 64 tile on or below the
// diagonal: it reads the tile of H64 along its rows, writes it to H, and writes the mirrored tile from LDS, so that both
// the reads and the writes run along rows.  The tile's loads are in flight together (one at a time a single tile took 8 us).
// RIDGE: lam = lambda_abs + lambda_rel trace / d1 first, by every workgroup for itself (d1 loads; the first leaves it in *ridge):
// for small layers, whose time is launches; *clear = 0 for a launch behind it.
template <bool RIDGE>
__global__ __launch_bounds__(256) void finalize_H_kernel(const double* __restrict__ H64, float* __restrict__ H, int d1,
                                                          const double* __restrict__ lam_dev, double lambda_abs, double lambda_rel, double* __restrict__ ridge,
                                                          int* __restrict__ clear) {
  __shared__ float tile[64][65];
  __shared__ double sh[4], s_lam;
  // tile index -> (tr, tc), tc <= tr
  const int t = blockIdx.x;
  int tr = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((int64_t)(tr + 1) * (tr + 2) / 2 <= t) tr++;
  while ((int64_t)tr * (tr + 1) / 2 > t) tr--;
  const int tc = t - tr * (tr + 1) / 2;
  const int r0 = tr * 64, c0 = tc * 64;
  const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;
  double x[16];
#pragma unroll
  for (int k = 0; k < 16; k++) {
    // on a diagonal tile the entries above the diagonal come from their mirror images
    const int i = min(r0 + ly + 4 * k, d1 - 1), j = min(c0 + lx, d1 - 1), hi = max(i, j), lo = min(i, j);
    x[k] = H64[(int64_t)hi * d1 + lo];
  }
  double lam;
  if constexpr (RIDGE) {
    double v = 0;
    for (int i = threadIdx.x; i < d1; i += 256) v += H64[(int64_t)i * d1 + i];
    v = block_sum(v, sh);
    if (threadIdx.x == 0) {
      s_lam = lambda_abs + lambda_rel * v / (double)d1;
      if (t == 0) { *ridge = s_lam; if (clear) *clear = 0; }
    }
    __syncthreads();
    lam = s_lam;
  } else {
    lam = lam_dev ? lam_dev[0] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int i = r0 + ly + 4 * k, j = c0 + lx;
    const float v = (float)(i == j ? x[k] + lam : x[k]);
    if (i < d1 && j < d1) H[(int64_t)i * d1 + j] = v;
    tile[ly + 4 * k][lx] = v;
  }
  if (tr == tc) return;
  __syncthreads();
  for (int k = 0; k < 16; k++) {
    const int i = c0 + ly + 4 * k, j = r0 + lx;      // row of the mirrored tile, column along the lanes
    if (i < d1 && j < d1) H[(int64_t)i * d1 + j] = tile[lx][ly + 4 * k];
  }
}

hipError_t launch_finalize_H(const double* H64, float* H, int d1, const double* lam_dev, hipStream_t s) {
  const int64_t nt = (d1 + 63) / 64;
  hipLaunchKernelGGL(finalize_H_kernel<false>, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, s, H64, H, d1, lam_dev, 0.0, 0.0, (double*)nullptr, (int*)nullptr);
  return hipGetLastError();
}
hipError_t launch_finalize_ridge(const double* H64, float* H, int d1, double lambda_abs, double lambda_rel, double* ridge, hipStream_t s, int* clear) {
  const int64_t nt = (d1 + 63) / 64;
  hipLaunchKernelGGL(finalize_H_kernel<true>, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, s, H64, H, d1, (const double*)nullptr, lambda_abs,
                     lambda_rel, ridge, clear);
  return hipGetLastError();
}

__global__ __launch_bounds__(1024) void trace64_kernel(const double* __restrict__ H64, int d1, double* out) {
  __shared__ double sh[16];
  double v = 0;
  for (int i = threadIdx.x; i < d1; i += blockDim.x) v += H64[(int64_t)i * d1 + i];
  double t = block_sum(v, sh);
  if (threadIdx.x == 0) out[0] = t;
}

hipError_t launch_trace64(const double* H64, int d1, double* out, hipStream_t s) {
  hipLaunchKernelGGL(trace64_kernel, dim3(1), dim3(1024), 0, s, H64, d1, out);
  return hipGetLastError();
}

// norms2[j] = sum of squares of the q rows of group j (one workgroup per group, fixed order, eight loads in flight: with 256
// threads and one load at a time 64 groups of 64 x 4096 took 0.28 ms)
__global__ __launch_bounds__(1024) void group_norms_kernel(const float* __restrict__ Wf, int q, int m,
                                                            double* __restrict__ norms2) {
  __shared__ double sh[16];
  const int g = blockIdx.x, nt = blockDim.x;
  const float* base = Wf + (int64_t)g * q * m;
  const int64_t n = (int64_t)q * m;
  double v = 0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < n; i += nt) { const double x = base[i]; v += x * x; }
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) norms2[g] = t;
}

hipError_t launch_group_norms(const float* Wf, int p, int q, int m, double* norms2, hipStream_t s) {
  hipLaunchKernelGGL(group_norms_kernel, dim3(p), dim3((int64_t)q * m >= 16384 ? 1024 : 256), 0, s, Wf, q, m, norms2);
  return hipGetLastError();
}

// out = sum a[i]*b[i] in float64, two fixed-order stages (partial must hold 1024 doubles)
__global__ __launch_bounds__(256) void dot64_stage1(const float* __restrict__ a, const float* __restrict__ b, int64_t n,
                                                     double* __restrict__ partial) {
  __shared__ double sh[4];
  double v = 0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) v += (double)a[i] * (double)b[i];
  double t = block_sum(v, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}
__global__ __launch_bounds__(1024) void dot64_stage2(const double* __restrict__ partial, int n, double* out) {
  __shared__ double sh[16];
  double v = (threadIdx.x < (unsigned)n) ? partial[threadIdx.x] : 0.0;
  double t = block_sum(v, sh);
  if (threadIdx.x == 0) out[0] = t;
}

// out = sum_i <a[rows[i], :], b[i, :]> (a: row-major with leading dimension m, b: dense nrows x m), float64, fixed order
__global__ __launch_bounds__(256) void dot64_rows_stage1(const float* __restrict__ a, const int32_t* __restrict__ rows,
                                                          const float* __restrict__ b, int nrows, int m, double* __restrict__ partial) {
  __shared__ double sh[4];
  double v = 0;
  for (int i = blockIdx.x; i < nrows; i += gridDim.x) {
    const float* ar = a + (int64_t)rows[i] * m;
    const float* br = b + (int64_t)i * m;
    for (int c = threadIdx.x; c < m; c += 256) v += (double)ar[c] * (double)br[c];
  }
  double t = block_sum(v, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}
hipError_t launch_dot64_rows(const float* a, const int32_t* rows, const float* b, int nrows, int m, double* out, double* partial,
                             hipStream_t s) {
  hipLaunchKernelGGL(dot64_rows_stage1, dim3(1024), dim3(256), 0, s, a, rows, b, nrows, m, partial);
  hipLaunchKernelGGL(dot64_stage2, dim3(1), dim3(1024), 0, s, partial, 1024, out);
  return hipGetLastError();
}

__global__ __launch_bounds__(1024) void sumsq_add_kernel(const double* __restrict__ part, double* __restrict__ acc) {
  __shared__ double sh[16];
  double t = block_sum(part[threadIdx.x], sh);
  if (threadIdx.x == 0) acc[0] += t;
}

hipError_t launch_dot64(const float* a, const float* b, int64_t n, double* out, double* partial, hipStream_t s) {
  hipLaunchKernelGGL(dot64_stage1, dim3(1024), dim3(256), 0, s, a, b, n, partial);
  hipLaunchKernelGGL(dot64_stage2, dim3(1), dim3(1024), 0, s, partial, 1024, out);
  return hipGetLastError();
}

}  // namespace osscar
