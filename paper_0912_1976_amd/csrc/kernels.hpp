// Device kernels of the PCG hot path (gfx950, wave64) and their launchers.
// All launchers enqueue on the given stream and never synchronise.
//
// Every vector kernel works on K right-hand sides at once (K in {1,2,4,8}):
// vectors are stored row-major as [n][K], so a matrix entry is read once
// for all K columns and the K values of a gathered row are contiguous.
// The vector type T is double (FP64 path) or float (inner solve of the
// mixed-precision path); reductions always accumulate in double.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vemg {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kSlicesPerBlock = kBlock / kWave;
constexpr int kMaxBatch = 8;

// SELL-64 matrix: 64 consecutive rows form a slice stored column-major and
// padded to the slice's longest row, so lane t of a wavefront reads entry k
// of row 64 s + t at sptr[s] + 64 k + t (coalesced).  Only off-diagonal
// entries are stored; padding entries have value 0 and point at the row
// itself (square) or column 0 (rectangular).
//   fine A (difference form): FP64 values a_ij with the deficit d64;
//   FP32 copy: row-scaled values a_ij / a_ii with s32 = a_ii and
//   dh32 = d_i / a_ii, so (A x)_i = s_i (sum_j w_ij (x_j - x_i) + dh_i x_i).
// The fine A holds in every row first the couplings to earlier sweep colours
// (the lower part L of its multicolour order), then those to later ones (U);
// in slice s the L entries end at smid[s], each part padded to the slice's
// longest.  The forward sweep from zero reads L alone and the residual after
// it U alone (sell_span).
struct Sell {
  const int64_t *sptr = nullptr;  // nslices + 1 entry offsets
  const int64_t *smid = nullptr;  // fine A: where slice s's U entries begin
  const int32_t *col = nullptr;
  const int32_t *col2 = nullptr;  // rows over the difference of two vector rows (MergedRows::top): the second, or -1
  const double *val64 = nullptr;
  const float *val32 = nullptr;
  const double *d64 = nullptr, *i64 = nullptr;  // deficit d_i and 1 / a_ii
  const float *s32 = nullptr, *dh32 = nullptr;
  int64_t nrows = 0;
};

// A slice in a visit order: its number and where its entries, its U entries
// and its end are (sptr, smid and the next sptr, in one load)
struct SliceRef {
  int64_t slice, begin, mid, end;
};

// CSR matrix (coarse multigrid operators, restrictions, coarse prolongators):
// a row's entries are dealt in turn to G groups of lanes (a power of two
// chosen from the mean row length), each group holding the row's K columns 16
// bytes a lane, and the groups' sums are added across lanes.  Square
// operators store off-diagonals only: FP64 values; FP32 values a_ij / a_ii
// with s32 = a_ii; row i's entries with columns > i (later in the sweep order)
// begin at upper[i].
struct CsrG {
  const int32_t *ptr = nullptr;  // nrows + 1
  const int32_t *upper = nullptr;
  const int32_t *col = nullptr;
  const double *val64 = nullptr;
  const float *val32 = nullptr;
  const float *s32 = nullptr;
  // rectangular operators only: stored row i is output row orow[i] (the rows
  // are stored in the spatial order of the columns they gather); null: i
  const int32_t *orow = nullptr;
  int64_t nrows = 0;
  int G = 4;
};

// Device scalars of one batched PCG solve (one set per column).
struct Scal {
  double rho[kMaxBatch], alpha[kMaxBatch], beta[kMaxBatch], bnorm2[kMaxBatch], rr[kMaxBatch],
      pq[kMaxBatch];
  double tol2[kMaxBatch];  // squared relative tolerance of each column
  int done[kMaxBatch], iters[kMaxBatch], status[kMaxBatch];  // status: 0 running, 1 converged,
                                                            // 2 max_iter, -6 breakdown
  int maxit[kMaxBatch];  // iteration cap of each column
  int all_done, K;
};

// Stopping parameters of the slots that (re)start in a continuous batch:
// each column converges on its own request's tolerance and iteration cap.
struct SlotStop {
  double tol[kMaxBatch];
  int maxit[kMaxBatch];
};

inline int64_t sell_blocks(int64_t r0, int64_t r1) {
  if (r1 <= r0) return 0;
  int64_t s0 = r0 / kWave, s1 = (r1 + kWave - 1) / kWave;
  return (s1 - s0 + kSlicesPerBlock - 1) / kSlicesPerBlock;
}
inline int64_t vec_blocks(int64_t n) { return (n + kBlock - 1) / kBlock; }

// ---- fine matrix (SELL, difference form) ---------------------------------
// y = A x (mode 0) on rows [r0, r1), or the residual y = g - A x right after a
// forward multicolour Gauss-Seidel sweep from zero with relaxation 1 that gave
// x (mode 1): (L + D) x = g, so g - A x = -U x and g is not read.  With
// partial, partial[block * K + k] = sum over the block's rows of x_ik y_ik.
// order: the range's slices in visit order, such that the blocks of one XCD
// take one spatial region of every colour.
template <class T>
void launch_spmv(hipStream_t st, int K, const Sell &A, int mode, int64_t r0, int64_t r1, const T *x, T *y,
                 double *partial, const int *done, const SliceRef *order);
// One multicolour Gauss-Seidel step on the rows [a0,a1) and [b0,b1) (rows of
// one colour): x_i += (g_i - (A x)_i) / a_ii.  first: the first sweep from
// x = 0, in ascending colours, x_i = (g_i - (L x)_i) / a_ii; x needs no fill.
// With dot: dot[block * K + k] = sum over the block's rows of g_ik x_ik (the
// updated x; a backward sweep updates every row once, so its colours together
// give g . x).  Returns the number of blocks.
template <class T>
int64_t launch_gs(hipStream_t st, int K, const Sell &A, int64_t a0, int64_t a1, int64_t b0, int64_t b1, const T *g,
                  T *x, const int *done, bool first, double *dot = nullptr);

// VL + additive smoother in one pair of fine sweeps.  The preconditioner is
// the sum of the SOR cycle (x) and the smoother's cycle on the non-top rows
// (u, zero on the top), two cycles of one matrix and one right-hand side g:
//   forward from zero: u = x except on the "dirty" rows D, the non-top rows
//     with a top row or a dirty row among their neighbours of earlier colours;
//   residual -U x: the smoother's differs only on the rows R with a top or a
//     dirty row among their neighbours of later colours;
//   backward: w = x + u (x on the top) obeys the sweep of the whole matrix
//     with right-hand side 2 g on the non-top rows and g on the top; a top row
//     needs its non-top neighbours' x = w - u, and the u of those
//     neighbours, followed through the sweep, needs u on D, with old values
//     on R: the same two sets.
// So one sweep serves both cycles, and beside it only u on X = D + R is
// carried, as nx more rows of the same vectors (row n + p for the p-th row of
// X, those of D first and in colour order).
struct MergedRows {
  int64_t n = 0, n_top = 0, nd = 0, nr = 0, nx = 0;
  const int32_t *drow = nullptr;  // D: matrix row of each
  const int32_t *rpos = nullptr;  // R: position in X of each
  const int32_t *xpos = nullptr;  // matrix row -> position in X, or -1
  Sell fwd;   // D rows, couplings to non-top rows of earlier colours (columns of the extended vector)
  Sell res;   // R rows, couplings to non-top rows of later colours
  Sell bwd;   // D rows, couplings to all non-top rows; the deficit includes the top couplings
  Sell top;   // top rows: column and, for non-top neighbours, their extended row (col2)
  Sell prol;  // [E~ | P0]: columns < n_top of the surface vector, then those of A_bar's first coarse level
};
// One colour of the two cycles' forward (first) or backward sweep: the rows
// [a0,a1) (top), [b0,b1) (non-top) and D's [d0,d1); dot as in launch_gs, over
// the matrix's rows.
template <class T>
int64_t launch_gs_merged(hipStream_t st, int K, const Sell &A, const MergedRows &M, int64_t a0, int64_t a1, int64_t b0,
                         int64_t b1, int64_t d0, int64_t d1, const T *g, T *x, const int *done, bool first,
                         double *dot = nullptr);
// y = -U x on every row, and on R's extended rows.
template <class T>
void launch_res_merged(hipStream_t st, int K, const Sell &A, const MergedRows &M, const T *x, T *y, const int *done,
                       const SliceRef *order);
// Between the sweeps: x = x + E~ ys on the top; below it w = (x + E~ ys) +
// (u + P0 ya), with u + P0 ya stored on X's extended rows.
template <class T>
void launch_prolong_merged(hipStream_t st, int K, const MergedRows &M, const T *ys, const T *ya, T *x,
                           const int *done);
// y = E x (accumulate: y += E x) for a rectangular SELL matrix, rows [0, nrows).
template <class T>
void launch_rect(hipStream_t st, int K, const Sell &E, bool accumulate, const T *x, T *y, const int *done);
// z_i = (E~ y)_i + (i >= n_top ? w_i : 0); partial[block * K + k] = sum r_ik z_ik.
template <class T>
void launch_prolong_sum(hipStream_t st, int K, const Sell &E, int64_t n_top, const T *y, const T *w, const T *r,
                        T *z, double *partial, const int *done);

// ---- coarse operators and transfers (CsrG) -------------------------------
// The coarse operations take one or two jobs a launch: the surface and the
// A_bar hierarchy are independent, their levels are too small to fill the
// chip, and a launch costs as much for one as for both.
// kCsrUpper: y = -U x, the residual g - A x right after a forward sweep from
// zero that gave x (square); kCsrMult: y = P x; kCsrAdd: y += P x
enum CsrMode { kCsrUpper, kCsrMult, kCsrAdd };
template <class T>
struct CsrJob {
  CsrG A;
  const T *x = nullptr;
  T *y = nullptr;
};
template <class T>
void launch_csr(hipStream_t st, int K, CsrMode mode, const CsrJob<T> *jobs, int nj, const int *done);
// Block multicolour (patch) order of a coarse level: its unknowns are stored
// patch by patch (patch colour, patch, local colour), a patch holding at most
// kPatchLdsRows unknowns.  Unknowns of patches of one colour are never
// coupled, so a forward sweep is, patch colour by patch colour, one exact
// triangular solve per patch: with h_p = g_p - A_pq x_q over the couplings
// to other patches (and to the patch's own later unknowns, with their old
// values), the patch's new values are (D_p + L_p)^{-1} h_p, L_p the strictly
// lower part of the patch's block in stored order -- the sequential SOR
// sweep in that order.  Backward: (D_p + U_p)^{-1} = ((D_p + L_p)^{-1})^T.
constexpr int kPatchLdsRows = 128;
constexpr int kPatchTile = 16;
constexpr int kPatchHalo = 1024;
// stored patch: its first row, its number of rows m, where its factor tiles
// begin; its halo, the rows of other patches it is coupled to, ascending
// (those of earlier patches first), at most kPatchHalo of them listed; and the
// patches it is coupled to, likewise
struct PatchDesc {
  int32_t row0, m;
  int64_t toff;
  int32_t halo, nearly, nhalo;
  int32_t nbr, nbr_early, nbr_all;
};
// A row's entries (columns ascending, so in sweep order) by what a sweep of
// its patch takes: [b, own) earlier patches, [own, late) its own patch before
// the row, [late, next) its own patch after it, and from next on later patches
struct PatchRow {
  int32_t b, own, late, next;
};
struct PatchSweep {
  const PatchDesc *desc = nullptr;
  const PatchRow *rows = nullptr;  // [patch][kPatchLdsRows + 1]; row m holds the end of row m - 1's entries
  const int32_t *halo = nullptr;
  // column of each entry of the level's CsrG: the row in its own patch, or
  // kPatchLdsRows + its place in the halo, or ~column beyond the halo's list
  const int32_t *lcol = nullptr;
  const int32_t *nbr = nullptr;
  // FP64: F = (D_p + L_p)^{-1}; FP32 (row-scaled operator): F D_p, rounded;
  // tb: the same of F^T.  Tiles of 16 x 16, zero beyond m, tile row I (of
  // t = ceil(m / 16)) holding its tiles J <= I (tb: J >= I) in order from tile
  // I (I + 1) / 2 (tb: I t - I (I - 1) / 2); a tile stores for s = 0..3 and
  // lane l entry (l % 16, 4 s + l / 16), the operand order of the 16x16x4
  // matrix instructions.
  const double *tf64 = nullptr, *tb64 = nullptr;
  const float *tf32 = nullptr, *tb32 = nullptr;
};
// One Gauss-Seidel sweep over all the patches of a level, one block per patch,
// in ascending (kPatchBackward: descending) order of the patch colours.
// kPatchFirst: the forward sweep from x = 0, which reads of the other patches
// only those swept before, so x needs no fill.
enum PatchDir { kPatchFirst, kPatchForward, kPatchBackward };
template <class T>
struct PatchJob {
  CsrG A;
  PatchSweep S;
  int64_t np = 0;
  const T *g = nullptr;
  T *x = nullptr;
  // Progress of the level's sweeps: the patches begun in all launches so far
  // (np of them a launch, so begun / np numbers the launch), and for every
  // patch the number, from 1, of the last launch that has finished it.
  unsigned long long *begun = nullptr;
  unsigned *ended = nullptr;
};
template <class T>
void launch_patch_gs(hipStream_t st, int K, PatchDir dir, const PatchJob<T> *jobs, int nj, const int *done);
// x = Cinv g (dense m x m FP64, symmetric, row-major), K columns; part:
// dense_chunks(m) * m * K doubles of scratch for the column chunks' partial sums.
constexpr int kDenseChunk = 512;
inline int64_t dense_chunks(int64_t m) { return (m + kDenseChunk - 1) / kDenseChunk; }
template <class T>
struct DenseJob {
  const double *C = nullptr;
  int64_t m = 0;
  const T *g = nullptr;
  T *x = nullptr;
  double *part = nullptr;
};
template <class T>
void launch_dense(hipStream_t st, int K, const DenseJob<T> *jobs, int nj, const int *done);

// ---- vectors ([n][K]) ----------------------------------------------------
template <class T>
void launch_fill(hipStream_t st, T *x, int64_t count, T v, const int *done);
template <class T>
void launch_copy(hipStream_t st, const T *a, T *b, int64_t count, const int *done);
// partial[block * K + k] = sum a_ik b_ik
template <class T>
void launch_dot(hipStream_t st, int K, const T *a, const T *b, int64_t n, double *partial, const int *done);
// z_i += w_i for rows i >= row0; partial[block * K + k] = sum r_ik z_ik (updated z)
template <class T>
void launch_add_dot(hipStream_t st, int K, const T *w, const T *r, T *z, int64_t row0, int64_t n, double *partial,
                    const int *done);
template <class T>
void launch_jacobi(hipStream_t st, int K, const T *r, const double *diag, T *z, int64_t n, const int *done);
// natural <-> storage order for column k of a batch (stride K)
void launch_gather(hipStream_t st, int K, int k, const double *nat, const int64_t *perm, double *sto, int64_t n);
void launch_scatter(hipStream_t st, int K, int k, const double *sto, const int64_t *perm, double *nat, int64_t n);
// the first cols columns of a batch, natural [cols][N] <-> storage [n][K] (the
// others 0); pos: storage row of each of the N nodes, -1 (value 0) if fixed
void launch_gather_batch(hipStream_t st, int K, const double *nat, int64_t N, const int64_t *perm, double *sto,
                         int64_t n, int cols);
void launch_scatter_batch(hipStream_t st, int K, const double *sto, const int32_t *pos, double *nat, int64_t N,
                          int cols);
// mixed precision: r32 = r64 * scale[k];  x64 = scale[k] * d32
void launch_demote(hipStream_t st, int K, const double *r64, const double *scale, float *r32, int64_t n,
                   const int *done);
void launch_promote(hipStream_t st, int K, const float *d32, const double *scale, double *x64, int64_t n,
                    const int *done);

// z64 = scale[k] z32; partial[block * K + k] = sum r_ik z_ik
void launch_promote_dot(hipStream_t st, int K, const float *z32, const double *scale, const double *r, double *z64,
                        int64_t n, double *partial, const int *done);

// ---- PCG scalars (partials are summed in index order) --------------------
// From kCompactFrom rows of partials on, launch_compact first adds them in
// kCompact consecutive parts, one block each (a single block takes 14 us for
// 8514 rows of 8 columns).
constexpr int64_t kCompactFrom = 4096;
constexpr int kCompact = 64;
void launch_compact(hipStream_t st, int K, const double *p, int64_t np, double *out, const int *done);
// with scale_in: scale_in[k] = 1 / ||b_k||, scale_out[k] = ||b_k|| (0 unless finite and positive)
void launch_pcg_init(hipStream_t st, int K, Scal *s, const double *pb, int64_t npb, double tol, int maxit,
                     double *scale_in = nullptr, double *scale_out = nullptr);
void launch_pcg_set_rho(hipStream_t st, int K, Scal *s, const double *p, int64_t np);
// The scalars alternate between two records: `in` as the iteration finds them,
// `mid` after alpha (and the convergence test).
// Folded: launch_pcg_xr takes the partials of p.q and forms alpha,
// launch_pcg_p those of r.z and forms beta, and with those of r.r applies the
// convergence test too; every block adds the partials, the first one writes
// the record.  A launch of one block took 4 to 5 us in their place.  The test
// folded into launch_pcg_p comes after the preconditioner, whose application
// in the iteration that converges is then for nothing, and every block adds
// the partials of r.r too.  Time of a solve with the test folded against a
// launch of its own, on one handle at 2600 to 255,024 unknowns: one column
// 0.995 to 1.013, eight 1.002 to 1.034; 113 x 105 x 21 with two columns 0.99,
// 25 x 25 x 17 mixed with four 0.99.  Above, one column at 330,749 to 515,624
// 0.991 to 1.003 and at 752,432 1.006 to 1.012 (eight do not fold).  The line
// (kFoldConvMax unknowns) bounds what the wasted application costs.
// Otherwise launch_pcg_alpha (in -> mid), launch_pcg_conv (mid) and
// launch_pcg_beta (mid -> in) do so in single blocks.
struct PartialSums {
  const double *p = nullptr;  // [n][K]; null: not folded
  int64_t n = 0;
};
// whether an iteration on n rows with K columns folds (np: rows of partials of
// its longest sum)
inline bool pcg_folds(int64_t np, int K) { return np <= kCompactFrom && np * K <= 8192; }
constexpr int64_t kFoldConvMax = 250000;
void launch_pcg_alpha(hipStream_t st, int K, const Scal *in, Scal *mid, PartialSums pq);
// x += alpha p, r -= alpha q, partial sums of r.r; with r32: r32 = scale r
template <class T>
void launch_pcg_xr(hipStream_t st, int K, const Scal *in, Scal *mid, PartialSums pq, T *x, T *r, const T *p,
                   const T *q, int64_t n, double *partial, float *r32, const double *scale);
void launch_pcg_conv(hipStream_t st, int K, Scal *mid, PartialSums rr);
void launch_pcg_beta(hipStream_t st, int K, const Scal *mid, Scal *in, PartialSums rz);
// p = z + beta p
template <class T>
void launch_pcg_p(hipStream_t st, int K, const Scal *mid, Scal *in, PartialSums rr, PartialSums rz, T *pvec,
                  const T *z, int64_t n);
// out[k] = sum of the partials of column k
void launch_reduce(hipStream_t st, int K, const double *p, int64_t np, double *out);
// before a restart: clears done/status of the columns whose bit in keep is 0
void launch_pcg_resume(hipStream_t st, int K, Scal *s, unsigned keep);

// ---- extended iterate across restarts (refine.hip) ----------------------
// The solution is the unevaluated sum hi + lo ([n][K] each); a restart's
// correction x is folded in without rounding error for the columns in mask
// (hi + x rounded, its error added to lo; x = 0 afterwards).
void launch_fold(hipStream_t st, int K, unsigned mask, double *hi, double *lo, double *x, int64_t n);
// res = b - A (hi + lo) on the fine difference-form matrix, with error-free
// products and double-double sums, rounded once (K in {1,2,4,8}).
void launch_residual_ext(hipStream_t st, int K, const Sell &A, const double *b, const double *hi, const double *lo,
                         double *res);
// out = hi + lo (rounded), count entries
void launch_round(hipStream_t st, const double *hi, const double *lo, double *out, int64_t count);

// Continuous batching (K = kMaxBatch slots): columns in `mask` (re)start
// while the others keep their state.
//   join: hi_k = lo_k = x_k = 0, r_k = b_k;   restart: r_k = res_k (after a fold)
void launch_slot_vectors(hipStream_t st, unsigned mask, bool restart, const double *b, const double *res,
                         double *hi, double *lo, double *x, double *r, int64_t n);
// join: bnorm2_k from the partials of b.b, iters_k = 0; both: done_k = 0
// (1 for a zero right-hand side), status_k = 0, and the FP32 scaling of the
// preconditioner input scale_in_k = 1/||b_k||, scale_out_k = ||b_k||
void launch_slot_scalars(hipStream_t st, unsigned mask, bool restart, Scal *s, const double *pb, int64_t npb,
                         const SlotStop &stop, double *scale_in, double *scale_out);
// rho_k from the partials of r.z, for the columns in mask
void launch_slot_rho(hipStream_t st, unsigned mask, Scal *s, const double *p, int64_t np);
// p_k = z_k for the columns in mask
void launch_slot_copy(hipStream_t st, unsigned mask, const double *z, double *p, int64_t n);

}  // namespace vemg
