// Internal declarations shared by the translation units of libosscar (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <vector>

namespace osscar {

// message of the last failure of a call that takes no context, per host thread (returned by osscar_last_error(NULL))
void set_contextless_error(const char* msg);

// ----------------------------------------------------------------------------------------------
// gemm.hip : C = alpha * A * B + beta * Cin (+ diag_add on the diagonal), all row-major float32
// storage, products accumulated in float64 on the matrix cores (v_mfma_f64_16x16x4_f64).
// ----------------------------------------------------------------------------------------------
struct GemmArgs {
  int M, N, K;
  const float* A; int64_t lda;   // M x K
  const float* B; int64_t ldb;   // K x N
  const float* Cin; int64_t ldcin;  // M x N or nullptr (treated as zero)
  void* C; int64_t ldc;          // M x N, float or double
  double alpha, beta, diag_add;
  int c_is_f64;                  // output (and Cin) element type: 0 float, 1 double
  int lower_only;                // 1: compute only tiles that touch the lower triangle (row >= col)
  int trans_b;                   // 1: B is given as N x K row-major (C = alpha * A * B^T + ...)
  int acc_f32;                   // 1: accumulate in float32 (v_mfma_f32_32x32x2_f32); float32 output only
  // hints for the int8-digit product only (i8gemm.hip; any other kernel ignores them): A (B) is square with a diagonal far
  // above the rest of its rows (columns), to be kept out of the fixed-point digits and added in float64
  int i8_diag_a, i8_diag_b;
  // and a levelling of the contraction index: A is used as A 2^(ksign kexp[k]), B as 2^(-ksign kexp[k]) B (nullptr: none)
  const int* i8_kexp; int i8_ksign;
  // workspace of the 64 x 64 kernel (gemm64.hip) for the partial tiles of a cut contraction (nullptr: it never cuts)
  double* ws; size_t ws_bytes;
};
hipError_t launch_gemm_f64acc(const GemmArgs& a, hipStream_t s);
// diagnostic log of the launches above: enable (1) / disable and clear (0); read = rows of {M, N, K, kind, ms} with
// kind = 1 float32 accumulation | 2 float64 output | 4 lower triangle only | 8 B transposed; returns the number of rows
// kind also carries 16 = the int8-digit product of i8gemm.hip
void gemm_log_enable(int on);
int gemm_log_read(double* out, int capacity);
void gemm_log_open(int M, int N, int K, int kind, hipStream_t s, int* slot);
void gemm_log_close(int slot, hipStream_t s);

// ----------------------------------------------------------------------------------------------
// gemm64.hip : the same product in 64 x 64 tiles, the contraction cut into ranges where the tiles alone do not fill the chip,
// and from operands as the caller holds them
// ----------------------------------------------------------------------------------------------
// ROW: result rows x K, float32.  K_*: K x result rows, contraction along the rows.
enum Opk64 { OPK_ROW_F32 = 0, OPK_K_F32 = 1, OPK_K_BF16 = 2 };
struct Gemm64 {
  int M, N, K, a_kind, b_kind, lower;
  const void* A; int64_t lda; const void* B; int64_t ldb;
  const void* Cin; int64_t ldcin; void* C; int64_t ldc; int c_is_f64;
  double alpha, beta, diag_add;
  double* ws; size_t ws_bytes;                // partial tiles of a cut contraction (none: never cut)
  const int *panels_m, *panels_n;             // set (never cut then): only the tiles in a marked panel of 128 rows or columns
};
constexpr size_t GEMM64_TILE_BYTES = 64 * 64 * 8;
hipError_t launch_gemm64(const Gemm64& q, hipStream_t s);
hipError_t launch_gemm64_logged(const Gemm64& q, hipStream_t s);      // with an entry in the log above: for callers outside gemm.hip

// ----------------------------------------------------------------------------------------------
// i8gemm.hip : the same product C = alpha A B + beta Cin (+ diag_add on the diagonal; lower_only) for float32 A, B, Cin, C
// with the accuracy of float64 accumulation, computed on the int8 matrix cores from I8_S seven-bit digits per operand
// ----------------------------------------------------------------------------------------------
constexpr int I8_S = 5, I8_S_BF16 = 4;
size_t i8_pack_bytes(int64_t rows, int64_t K);          // packed size of an operand with `rows` rows (A) or columns (B)
bool i8_gemm_fits(const GemmArgs& g);
// H64 += X^T X (lower triangle) and, with Y, G64 += X^T Y for K <= 16384 rows of float32 or bf16 at any alignment, except the tiles
// of the 128-column panels that *flag_x / *flag_y mark (device, in `words`): those the caller adds.  pack_x / pack_y
// hold i8_gram_rows(bytes, ...) >= K rows, words: i8_gram_word_bytes, 8-byte aligned
int64_t i8_gram_rows(size_t bytes, int x_bf16, int64_t cols);
size_t i8_gram_word_bytes(int64_t d1, int64_t m);
hipError_t launch_i8_gram(const void* X, int x_bf16, int64_t ldx, int d1, const void* Y, int64_t ldy, int m, int K, double* H64, double* G64,
                          void* pack_x, void* pack_y, unsigned* words, const int** flag_x, const int** flag_y, hipStream_t s);
// kexp[k] = round(log2 sqrt(D_kk)) from the diagonal of a Gram block (device, n ints)
hipError_t launch_i8_kexp(const float* D, int n, int64_t ld, int* kexp, hipStream_t s);
// packA / packB: scratch for the two packed operands (capacities in bytes), mx: M + N words for the scaling exponents
hipError_t launch_i8_gemm(const GemmArgs& g, void* packA, size_t capA, void* packB, size_t capB, unsigned* mx, size_t mx_entries,
                          hipStream_t s);

// ----------------------------------------------------------------------------------------------
// gram.hip : H64 (+)= Xc^T Xc on the lower-triangle tiles (bf16 X, d1 % 8 == 0, ldx % 8 == 0, 16-byte aligned)
// ----------------------------------------------------------------------------------------------
// Tile schedules of a packed product on the device, uploaded once by the caller (no call here waits for the stream): 128 x 128
// tiles (gram_tile_list_host / rect_tile_list_host) and, optionally, 256 x 192 tiles (wide_tile_list_host) and 256 x 128 tiles
// (tall_tile_list_host).
struct PackedTiles { const int2* list = nullptr; size_t entries = 0; const int2* wide = nullptr; size_t wide_entries = 0;
                     const int2* tall = nullptr; size_t tall_entries = 0; };
// A float64 result that is accumulated over calls, as the sum of up to `copies` consecutive copies of it; *cleared = how many of
// them hold something (or zeros) so far, nullptr: the caller has cleared all.
struct PackedAcc { double* out = nullptr; int copies = 1; int* cleared = nullptr; };
hipError_t launch_sum_copies(double* A, int copies, int rows, int cols, int lower, hipStream_t s);      // into the first one, in order
int packed_copies(int64_t elems, int64_t ntiles);      // copies worth keeping for a result of this many elements and 128 x 128 tiles
// Patch geometry of a convolutional layer: row (b*Hout + oy)*Wout + ox, column (c*kh + dy)*kw + dx of the patch matrix is
// F[b][c][oy*stride + dy - pad][ox*stride + dx - pad] (zero outside the map).
struct ConvSpec { int B, C, Hin, Win, kh, kw, stride, pad, Hout, Wout; };
// What waits in the pack buffers: stages of 64 rows, where the rows of a call end (a bit per pair of stages), the windows' length
struct PackQueue {
  int stages = 0, last = 0, calls = 0, window = 16, window_y = 16;      // last: stages of the last call's rows
  uint64_t ends[2] = {0, 0};
  int64_t rows = 0;
  int ev_used = 0; int64_t ev_rows = 0;      // event pairs recorded by the launches since the caller cleared them, rows of these launches
  void clear() { stages = calls = 0; window = window_y = 16; ends[0] = ends[1] = 0; rows = 0; }
};
// H64 += X^T X (lower triangle) and, with pack_y, G64 += X^T Y from bf16 rows.  pack_x: pack_stages (<= 256) * 64 rows of 128*ceil(d1/128)
// bf16, pack_y of 128*ceil(m/128).  ev (optional, 2 * ev_pairs events): recorded before and after launches of the symmetric product.
struct PackedGram {
  PackQueue* q;
  int d1; PackedAcc H64; PackedTiles tiles; void* pack_x;
  int m; PackedAcc G64; PackedTiles tiles_y; void* pack_y;
  int pack_stages; hipEvent_t* ev; int ev_pairs;
  double* spare; size_t spare_bytes;      // unused memory of the phase, for parts of the tiles that do not fill a round (may be none)
};
// Repacks rows into MFMA operand order and accumulates their products, at once or when the buffer is full; launch_gram_queue adds
// what still waits.  conv (optional): Xc is a feature map (NCHW, bf16) and the rows are its patches.
hipError_t launch_gram_packed(const PackedGram& g, const void* Xc, int64_t n_c, int64_t ldx, const void* Yc, int64_t ldy, const ConvSpec* conv,
                              hipStream_t s);
hipError_t launch_gram_queue(const PackedGram& g, hipStream_t s);
// host-side schedules: lower-triangle tiles of a d1 x d1 result / all tiles of a d1 x m result (128 x 128 tiles)
void gram_tile_list_host(int d1, std::vector<int2>& out);
void rect_tile_list_host(int d1, int m, std::vector<int2>& out);
// the same for the 256 x 192 tiles of a rows x cols result (symmetric: of its lower triangle)
void wide_tile_list_host(int rows, int cols, bool symmetric, std::vector<int2>& out);
void tall_tile_list_host(int rows, int cols, bool symmetric, std::vector<int2>& out);
size_t wide_tile_entries(int64_t rows, int64_t cols);      // an upper bound of that list's length
int gram_tile_schedule(int tiles_per_side, int32_t* out, int capacity);   // host only: the tile order of the SYRK kernel
// G64 (zeroed by the caller) += H W for bf16 W through three bf16 pieces of the float32 H (see gram.hip)
hipError_t launch_hw_split(const float* H, int d1, const void* W, int64_t ldw, int m, double* G64, const PackedTiles& tiles,
                           void* pack_h, void* pack_w, int64_t pack_rows, hipStream_t s);
// Products of float32 matrices on the bf16 matrix cores through three bf16 pieces per operand (see gram.hip).  Operands are
// row-major with the contraction along their rows (C = A^T B).  pack: split_pack_bytes(K, cols) bytes, 256-byte aligned.
size_t split_pack_bytes(int64_t K, int64_t cols);
hipError_t launch_pack_pieces(const float* A, int64_t lda, int64_t K, int cols, void* pack, hipStream_t s);   // cols % 8 == 0, lda % 4 == 0
// acc (M x N float64, dense; cleared here) = A^T B.  tiles: rect_tile_list_host(M, N), or gram_tile_list_host(M) for the lower
// triangle of a square result (ntiles = number of real tiles in the list)
hipError_t launch_split_product(const void* packA, int M, const void* packB, int N, int64_t K, int nprod, double* acc,
                                const PackedTiles& tiles, int ntiles, hipStream_t s);
// C = float(beta * Cin + alpha * acc)
hipError_t launch_split_epilogue(const double* acc, int M, int N, const float* Cin, int64_t ldcin, float* C, int64_t ldc, double alpha,
                                 double beta, hipStream_t s);
hipError_t launch_sumsq(const void* A, int is_bf16, int64_t rows, int64_t cols, int64_t ld, double* acc, double* partial,
                        hipStream_t s);   // partial: 1024 doubles
hipError_t launch_finalize_G(const double* G64, const float* Wf, const double* lambda_dev, float* G, int64_t n, hipStream_t s);
// H = float(mirror(H64) + lam*I); also usable with lam = 0
hipError_t launch_finalize_H(const double* H64, float* H, int d1, const double* lam_dev, hipStream_t s);
// the same with the ridge lambda_abs + lambda_rel trace / d1, which is left in *ridge (layers of up to RIDGE_DIM columns: every workgroup reads
// the diagonal; whole finalize with 16 columns of W, this way and with trace and ridge in launches of their own: 288 columns 35.5 / 39.3 us,
// 1024 42.9 / 46.6, 2048 56.4 / 57.4, 3072 98.6 / 91.3, 8192 575 / 320)
constexpr int RIDGE_DIM = 1024;
hipError_t launch_finalize_ridge(const double* H64, float* H, int d1, double lambda_abs, double lambda_rel, double* ridge, hipStream_t s, int* clear = nullptr);
// out[0] = sum_i H64[i][i]
hipError_t launch_trace64(const double* H64, int d1, double* out, hipStream_t s);
// rows r0 .. r0 + nr of the patch matrix as float32, nr x d1
hipError_t launch_im2col_rows(const void* F, int is_bf16, const ConvSpec& cs, int64_t r0, int64_t nr, int d1, float* out, hipStream_t s);
hipError_t launch_convert_to_f32(const void* src, int is_bf16, int64_t rows, int64_t cols, int64_t lds, float* dst,
                                 hipStream_t s);
// norms2[j] = sum over group j of W^2 (float64); c0 = sum W*G
hipError_t launch_group_norms(const float* Wf, int p, int q, int m, double* norms2, hipStream_t s);
hipError_t launch_dot64(const float* a, const float* b, int64_t n, double* out, double* partial, hipStream_t s);
// out = sum_i <a[rows[i], :], b[i, :]>, a with leading dimension m, b dense nrows x m (partial: 1024 doubles)
hipError_t launch_dot64_rows(const float* a, const int32_t* rows, const float* b, int nrows, int m, double* out, double* partial,
                             hipStream_t s);

// ----------------------------------------------------------------------------------------------
// tableau.hip : the swept tableau N (d1 x d1, lower triangle valid) and Z (d1 x m)
//   N_KK = -P, N_{K,Kc} = V, N_{Kc,Kc} = S (Schur complement), Z_K = B, Z_Kc = R.
// ----------------------------------------------------------------------------------------------
struct SearchCtrl {          // lives in device memory
  int32_t done;              // set when a swap is rejected (or nothing left to swap)
  int32_t iters;             // iterations run
  int32_t accepted;          // swaps applied
  int32_t notpd;             // a pivot block was not definite
  int32_t g_out, g_in;       // current selection (group ids), -1 if none
  int32_t pause;             // delayed-update search: the host must flush before the search can go on
  int32_t tau;               // delayed-update search: number of pending pivots that every kernel of an iteration works with
  int32_t tau_inc;           // pivots that the iteration just applied adds to it: folded into tau by the next one-workgroup
  int32_t misses;            // kernel (prep), so that no kernel changes tau while its own workgroups read it.
                             // misses: delayed-update search, pivots so far whose products with Z0 had not been computed ahead
  double obj;                // tracked objective
  double rel_tol;
  double delta;              // exact change of the current pair
  double gap_rem, gap_add;
  int32_t stalled;           // a run of swaps (swaprun.hip) waited too long and left everything as it was; runs behind it make no swap
  int32_t spare;             // one-launch swaps: spare slots of the look-ahead products in use (below zero: slots of picked rows are spare too)
  int32_t taken;             // groups: whether the pair of this iteration is taken, until the scores' launch records it
};

struct TabDims { int d1, m, p, q; };

hipError_t launch_gather(const float* src, int64_t lds, const int32_t* rows, int nrows, const int32_t* cols, int ncols,
                         float* dst, int64_t ldd, hipStream_t s);
// dst[rows[i]][cols[j]] = sign * src[i][j], only where rows[i] >= cols[j] if lower_only
hipError_t launch_scatter(const float* src, int64_t lds, const int32_t* rows, int nrows, const int32_t* cols, int ncols,
                          float* dst, int64_t ldd, float sign, int lower_only, hipStream_t s);
hipError_t launch_mirror_lower(float* A, int n, int64_t lda, hipStream_t s);
hipError_t launch_absmax(const float* A, int64_t n, double* out, hipStream_t s);

constexpr int INV_NB = 128;   // pivot block width of the sweep inverse
// In-place inverse of the symmetric positive definite n x n matrix A (full storage on entry and exit)
// by block sweeps of width INV_NB; panel/work buffers are caller-provided: panel (n*INV_NB), panelD (2*n*INV_NB),
// small (INV_NB*INV_NB doubles).  notpd_flag (device int) is set if a pivot block is not definite.
// The same with the working matrix in float64 (A64: n x n, panels: 4 n INV_NB float64): P = H^-1 rounded to float32 once.
// side (optional): a second stream with two events, on which the bulk of each panel's update runs beside the next panel's
// small kernels; every launch is joined back into s before the call returns.
struct SideStream;
hipError_t spd_inverse_f64(const float* H, int64_t ldh, int n, float* P, double* A64, double* panels, double* small,
                           int32_t* notpd_flag, hipStream_t s, const SideStream* side = nullptr);
hipError_t spd_inverse_inplace(float* A, int n, float* panel, float* panelD, double* small, int32_t* notpd_flag,
                               hipStream_t s);

struct TabPtrs {
  float* N; float* Z;              // tableau
  int32_t* kept;                   // p flags: 1 kept, 0 candidate
  double* score;                   // p scores: removal cost (kept) / addition gain (candidate)
  double* gram;                    // p * q*q : Z_g Z_g^T per group (float64)
  double* dblk;                    // p * q*q : float64 copy of the diagonal blocks N_gg
  float* C1; float* C2;            // d1 x q panels
  float* C1D; float* C2D;          // d1 x q panels times D
  float* rZ1; float* rZ2;          // q x m
  double* small;                   // scratch for q x q algebra (>= 16*q*q doubles)
  double* part;                    // group_part_doubles(): the column chunks of the groups' Grams (groups of more than one row)
  double* dpart;                   // ceil(m / 16) partial sums of the exact change of a pair (column blocks, fixed order)
  double* cross; double* xgram; double* xdblk; double* xscore;   // exact entering rule: d1*q, p*q*q, p*q*q, p
  SearchCtrl* ctrl;
  int32_t* trace_out; int32_t* trace_in; float* trace_gap; double* trace_obj;
};

size_t group_part_doubles(int64_t p, int64_t q, int64_t m);
hipError_t launch_refresh_scores(const TabDims& d, const TabPtrs& t, hipStream_t s);   // gram, dblk, score from N, Z
// ev (optional): three events recorded before the bulk update of N, after it, and after the update of Z.  Groups of
// more than one row: the one launch of both lies between the first two.
// single (optional, device): removal of the one group *single instead of a swap (Case 1 alone; no selection kernel).
// exact_in: the entering group is the argmax of the exact gain of the pair with the selected leaving group.
hipError_t launch_search_iteration(const TabDims& d, const TabPtrs& t, int forced_out, int forced_in, int always_accept,
                                   hipStream_t s, hipEvent_t* ev = nullptr, const int32_t* single = nullptr, int exact_in = 0);
// pick[0..take) = the kept groups of smallest removal cost (ascending), *gap = relative gap to the next one; take <= 64
// side 1: the groups outside the kept set with the largest addition gain (descending) instead; side 2: both in one launch,
// side 1's into pick + 64 and gap + 1
hipError_t launch_greedy_pick(const TabDims& d, const TabPtrs& t, int take, int32_t* pick, float* gap, hipStream_t s,
                              int side = 0);
hipError_t launch_select(const TabDims& d, const TabPtrs& t, int forced_out, int forced_in, hipStream_t s);

// ----------------------------------------------------------------------------------------------
// lazy.hip : delayed-update search for q = 1
// ----------------------------------------------------------------------------------------------
constexpr int LAZY_TM = 128;     // capacity of the pending pivot set (two per swap)
constexpr int LAZY_NC = 256;     // rows of Z0 whose products with all of Z0 are computed ahead, after every flush
constexpr int LAZY_NS = 64;      // spare slots for pivots that were not among them
constexpr int LAZY_NPICK_OUT = 88;  // swap search: kept rows picked by cost of removal ...
constexpr int LAZY_NPICK_IN = 72;   // ... and rows outside the kept set picked by gain; together a multiple of 32
constexpr int LAZY_BT = 16;      // rows that one block removal of the nested schedule takes at most
// best and second best score of a block of rows: [0] cheapest removal, [1] largest gain (negated); slot of the best row's products, -1 none
struct SwapRec { double best[2], second[2]; int32_t row[2], slot[2]; };
struct LazyPtrs {
  int32_t* pos;     // d1: position in the pending set or -1
  int32_t* Tidx;    // LAZY_TM pivot indices
  float* Jsg;       // LAZY_TM: -1 for pivots that left the kept set, +1 for pivots that entered
  float* C0R;       // d1 x LAZY_TM row-major: base columns N0[:, T_s]
  double* Minv;     // LAZY_TM x LAZY_TM: inverse of N0[T, T]
  double* ZT;       // LAZY_TM x m: Minv * Z0[T, :]
  float* ZT32;      // LAZY_TM x m (flush)
  float* E;         // d1 x LAZY_TM: C0 * Minv (flush)
  // products of Z0 with the rows of Z0 that are likely to become pivots before the next flush
  double* GbT;      // (LAZY_NC + LAZY_NS) x d1: row s = Z0 Z0[cand[s], :]^T
  double* rowsq;    // 2 ceil(m / 128) x d1: sums of squares of every row's 64-column stretches, left by Z0's update in the flush
  float* Zc;        // LAZY_NC x m: the gathered rows (shapes that take the general matrix-product kernel)
  // flush: E, C0 and ZT cut into three bf16 pieces in matrix-core operand order (768 bytes per padded row / column), and the
  // tile schedules of the two updates (the Gram kernel's: lower triangle of d1 x d1, all of d1 x m), uploaded at create
  void* Epk; void* Cpk; void* Zpk;
  const int2* tiles_sym; size_t n_tiles_sym; const int2* tiles_rect; size_t n_tiles_rect;
  double* gemm_ws; size_t gemm_ws_bytes;      // workspace of the 64 x 64 products (shapes that take the general kernels)
  void* ZcP;        // LAZY_NC x 32*ceil(m/32) x 3 bf16: the candidate rows cut into three bf16 pieces, in matrix-core operand order
  int32_t* cslot;   // d1: slot of a row in GbT or -1
  int32_t* cand;    // LAZY_NC + LAZY_NS: row held by a slot or -1
  int32_t* tslot;   // LAZY_TM: slot of each pending pivot
  // one-launch swaps (in the phases' scratch, see carve_all): the other copy of M^-1, two copies of a record per workgroup, Gram
  // matrix of the base rows in the slots (LAZY_NC + LAZY_NS squared) and its part for the pending pivots (LAZY_TM squared)
  double* Minv2; SwapRec* rec; SwapRec* rec2; double* K; double* KT;
  // runs of swaps: their shared words and two copies of ZT ZT^T for the pending pivots, where a flush has its packed operands (ZcP .. Zpk)
  void* run_shared; double* LL; double* LL2;
  double* lkey; int32_t* lidx;   // up to 2 x 1024: per-block winners of the candidate selection
  // block removal (nested schedule): X = M^-1 N0[T, G], U = ZT Y^T (LAZY_TM x LAZY_BT each), D, Y Y^T (LAZY_BT^2), the picks; the
  // removal lists of every 64 rows (in the phases' scratch)
  double* bX; double* bU; double* bD; double* bYY; int32_t* bG;
  double* lval; int32_t* lrow;
  int spare0;       // SearchCtrl::spare with nothing pending
};
// With no rows picked every pivot takes a spare slot: as many as can be pending (64 let the swaps flush after 32 instead of 64)
constexpr int spare_start(int mode) { return mode == 2 ? LAZY_NS - LAZY_TM : 0; }
// mode: which rows get their products with Z0 computed ahead: 0 = LAZY_NPICK_OUT cheapest removals + LAZY_NPICK_IN largest gains,
// 1 = LAZY_NC cheapest removals (removal-only loops), of every 1024 rows a side at most its share of 1024; 2 = none (every pivot then costs a pass over Z0)
hipError_t launch_lazy_init(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode = 0);
// Pairs on the device that swaps take in turn, out[r * step] and in[r * step] for r < n <= 64; in == nullptr: rows out[r * step] to remove
struct SwapList { const int32_t* out = nullptr; const int32_t* in = nullptr; int n = 0, step = 1; };
// swap.hip: one swap in one launch, from the control block t.ctrl, L.Minv and L.rec to *next, L.Minv2 and L.rec2 (the caller exchanges
// them after every launch); at most `limit` iterations will have run, the last l.n of them the list's; tau_most: at most this many pivots
// are pending.  A pivot whose products have not been computed ahead takes a launch of its own, which fetches them.
// fetch_only: it does nothing else.
hipError_t launch_lazy_swap(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, SearchCtrl* next, int always_accept, int limit, int tau_most,
                            hipStream_t s, const SwapList& l = SwapList(), bool fetch_only = false);
// swaprun.hip: the swaps up to `limit` iterations in one launch, between the same copies; it ends before a pivot whose products have not been
// computed ahead, which launch_lazy_swap then fetches.  run: number of the launch since the records were last refreshed, below RUN_MOST;
// patience: ticks of 10 ns that a workgroup waits for the others before all give up (SearchCtrl::stalled).  Lists: pairs only.
// The workgroups wait for one another, so all have to be resident at once (swap_run_fits); with a list they don't.  Their shared words are
// cleared with the records.  It takes ZT ZT^T from L.LL and leaves it in L.LL2 (exchanged after it, too), so all pending pivots have to come from runs.
constexpr int RUN_MOST = 64;
hipError_t launch_swap_run(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, SearchCtrl* next, int always_accept, int limit, int run, uint32_t patience,
                           hipStream_t s, const SwapList& l = SwapList());
bool swap_run_fits(int64_t d1);
constexpr int RUN_WGS = 256, RUN_WORDS = 5;                                                 // workgroups at most; words of a record's side
constexpr int RUN_SHARED_WORDS = 2 * 2 * RUN_WORDS * RUN_WGS + RUN_MOST;                     // the shared words of 64 bits
// Rows per workgroup: one workgroup per compute unit where the rows allow it (8192 = 256 x 32, 16384 = 256 x 64, 28672 = 224 x 128).
// More than 256 workgroups would run one after the other, and the algebra of order |T| is the same for each of them.
constexpr int swap_rows_per_wg(int d1) { return d1 <= 8192 ? 32 : d1 <= 16384 ? 64 : 128; }
int swap_record_count(int64_t d1);
hipError_t launch_swap_records(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, bool refresh);
hipError_t launch_cand_gram(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, int ncand, hipStream_t s);
hipError_t launch_zt(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s);
// `take` <= LAZY_BT rows leave the kept set as one block pivot (nested schedule, q = 1): those in pick (device), or (own_pick) the
// cheapest ones, which are left there, with the relative gap to the next one in *gap; at most tau_most pivots are pending.  Does nothing
// else but set ctrl->pause if a pick is pending, is not among the rows whose products were computed ahead, or the pending set
// has no room for all of them.
hipError_t launch_lazy_block_remove(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, int take, bool own_pick, int tau_most, int32_t* pick,
                                    float* gap, hipStream_t s);
int removal_list_count(int64_t d1);
hipError_t launch_removal_lists(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, bool refresh);

// A second stream and two events: the flush runs the candidate selection and its update of N0 there, beside the update of Z0 and the
// look-ahead product on the main stream (they touch disjoint data but for what the events order), and joins before the scores are refreshed.
struct SideStream { hipStream_t stream = nullptr; hipEvent_t fork = nullptr, join = nullptr; };
// side == nullptr (or no stream in it): everything in order on s
hipError_t launch_lazy_flush(const TabDims& d, const TabPtrs& t, const LazyPtrs& L, hipStream_t s, int mode = 0,
                             const SideStream* side = nullptr);

hipError_t launch_scatter_rows(const float* src, int64_t lds, const int32_t* rows, int nrows, int ncols, void* dst,
                               int64_t ldd, int dst_is_bf16, hipStream_t s);
hipError_t launch_fill_rows_zero(void* dst, int64_t ldd, int nrows_total, int ncols, int dst_is_bf16, hipStream_t s);

}  // namespace osscar
