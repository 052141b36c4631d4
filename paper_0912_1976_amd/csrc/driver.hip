// Solver handle: packs the host setup into HBM (SELL-64 fine operator,
// CSR for coarse operators and transfers, FP64 and FP32 copies), runs the
// preconditioned CG loop on the device for batches of up to eight right-hand
// sides, and exposes the C ABI of vemg.h.
//
// One PCG iteration is a fixed sequence of kernels on one stream whose scalars
// (alpha, beta, per-column convergence flags) live in device memory, so the
// chunk of iterations between two polls of the flags is captured once per
// (precision, batch width, length) in a hipGraph and replayed; every kernel
// returns at once when all columns have converged.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <numeric>
#include <thread>
#include <memory>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/vemg.h"
#include "kernels.hpp"
#include "setup.hpp"

namespace vemg {
namespace {

struct DeviceError : std::runtime_error {
  int code;
  DeviceError(int c, const std::string &m) : std::runtime_error(m), code(c) {}
};

#define HIPCHK(expr)                                                                              \
  do {                                                                                            \
    hipError_t e_ = (expr);                                                                       \
    if (e_ != hipSuccess)                                                                         \
      throw ::vemg::DeviceError(e_ == hipErrorOutOfMemory ? VEMG_ERR_OOM : VEMG_ERR_DEVICE,       \
                                std::string(#expr) + ": " + hipGetErrorString(e_));               \
  } while (0)

// device memory owned by a handle; with count_only set nothing is allocated or
// copied, only the bytes are added up (the footprint query).  All of it is one
// allocation: what an iteration reads of a mesh whose inverses nearly fill the
// Infinity Cache (71,824 unknowns, inverses of 210 MB) is kept there only if it
// lies together.  With an allocation per array its solve took 6.1 to 7.1 ms by
// what the process had allocated before, in one 6.0 to 6.6.
struct Arena {
  static constexpr size_t kAlign = 256;
  char *base = nullptr;
  size_t bytes = 0, reserved = 0;
  bool count_only = false;
  void reserve(size_t size) {
    HIPCHK(hipMalloc((void **)&base, size));
    reserved = size;
  }
  template <class T>
  T *alloc(size_t count) {
    const size_t at = bytes;
    bytes += (std::max<size_t>(count, 1) * sizeof(T) + kAlign - 1) / kAlign * kAlign;
    if (count_only) return nullptr;
    if (bytes > reserved) throw DeviceError(VEMG_ERR_DEVICE, "device allocations exceed the counted footprint");
    return (T *)(base + at);
  }
  template <class T>
  T *upload(const std::vector<T> &v, hipStream_t st) {
    T *p = alloc<T>(v.size());
    if (!v.empty() && !count_only) {
      // the source is a temporary host vector: finish the copy before returning
      HIPCHK(hipMemcpyAsync(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st));
      HIPCHK(hipStreamSynchronize(st));
    }
    return p;
  }
  void release() {
    if (base) (void)hipFree(base);
    base = nullptr;
    bytes = reserved = 0;
  }
};

// host copy of a Sell's sptr and smid
struct SellSpans {
  std::vector<int64_t> sptr, smid;
};

// fn(s) for every slice, on host threads by ranges of slices
template <class F>
void by_slices(int64_t ns, int64_t work, F &&fn) {
  parallel_threads(work, [&](int t, int nt) {
    for (int64_t s = ns * t / nt, s1 = ns * (t + 1) / nt; s < s1; ++s) fn(s);
  });
}

// the allocations of a Sell of n rows after its slice offsets, counted
Sell count_sell(Arena &ar, int64_t n, int64_t entries, bool pairs, bool data) {
  ar.alloc<int32_t>(entries);
  if (pairs) ar.alloc<int32_t>(entries);
  ar.alloc<double>(entries);
  ar.alloc<float>(entries);
  if (data) {
    ar.alloc<double>(n);
    ar.alloc<double>(n);
    ar.alloc<float>(n);
    ar.alloc<float>(n);
  }
  Sell M;
  M.nrows = n;
  return M;
}

// CSR (host) -> SELL-64 (device).  Square: the diagonal entries are taken
// out of the stored entries; the FP64 per-row term is `d` if given
// (difference form: the deficit) else a_ii.  FP32 copy: a_ij / a_ii with
// s32 = a_ii and dh32 = d / a_ii (square), or float(a_ij) (rectangular).
// colour (square): each row's couplings to earlier colours come first, then
// those to later ones, the two parts padded apart (Sell::smid).
Sell pack_sell(Arena &ar, hipStream_t st, const Csr &A, bool square, const std::vector<double> *d,
               const std::vector<double> *diag, int64_t *stored = nullptr,
               const std::vector<int32_t> *colour = nullptr, SellSpans *spans = nullptr) {
  int64_t n = A.nrows, ns = (n + kWave - 1) / kWave;
  // part of entry e of row r: 0 (earlier colour, or no colours) or 1; -1: not stored
  auto part_of = [&](int64_t r, int64_t e) {
    const int64_t c = A.idx[e];
    if (square && c == r) return -1;
    return colour && (*colour)[c] > (*colour)[r] ? 1 : 0;
  };
  std::vector<int64_t> sptr(ns + 1, 0), smid(ns, 0);
  by_slices(ns, A.nnz(), [&](int64_t s) {
    int64_t L[2] = {0, 0};
    for (int64_t r = s * kWave; r < std::min(n, (s + 1) * kWave); ++r) {
      int64_t len[2] = {0, 0};
      for (int64_t e = A.ptr[r]; e < A.ptr[r + 1]; ++e) {
        const int p = part_of(r, e);
        if (p >= 0) ++len[p];
      }
      for (int p = 0; p < 2; ++p) L[p] = std::max(L[p], len[p]);
    }
    smid[s] = L[0] * kWave;
    sptr[s + 1] = L[1] * kWave;
  });
  for (int64_t s = 0; s < ns; ++s) {
    smid[s] += sptr[s];
    sptr[s + 1] += smid[s];
  }
  if (stored) *stored = sptr[ns];
  if (spans) *spans = SellSpans{sptr, smid};
  if (ar.count_only) {
    ar.alloc<int64_t>(ns + 1);
    if (colour) ar.alloc<int64_t>(ns);
    return count_sell(ar, n, sptr[ns], false, square);
  }
  std::vector<int32_t> col(sptr[ns]);
  std::vector<double> val(sptr[ns], 0.0);
  std::vector<float> val32(sptr[ns], 0.0f);
  std::vector<double> dv(square ? n : 0, 0.0), ad(square ? n : 0, 0.0);
  for (int64_t r = 0; square && r < n; ++r) {
    if (diag) ad[r] = (*diag)[r];
    for (int64_t e = A.ptr[r]; e < A.ptr[r + 1]; ++e)
      if (A.idx[e] == r) ad[r] = A.val[e];
    dv[r] = d ? (*d)[r] : ad[r];
  }
  by_slices(ns, A.nnz(), [&](int64_t s) {
    for (int t = 0; t < kWave; ++t) {
      const int64_t r = s * kWave + t;
      int64_t pos[2] = {sptr[s] + t, smid[s] + t};
      for (int64_t e = r < n ? A.ptr[r] : 0; r < n && e < A.ptr[r + 1]; ++e) {
        const int p = part_of(r, e);
        if (p < 0) continue;
        col[pos[p]] = A.idx[e];
        val[pos[p]] = A.val[e];
        val32[pos[p]] = square ? (float)(A.val[e] / ad[r]) : (float)A.val[e];
        pos[p] += kWave;
      }
      const int64_t end[2] = {smid[s], sptr[s + 1]};
      for (int p = 0; p < 2; ++p)
        for (; pos[p] < end[p]; pos[p] += kWave) col[pos[p]] = (square && r < n) ? (int32_t)r : 0;
    }
  });
  Sell M;
  M.nrows = n;
  M.sptr = ar.upload(sptr, st);
  if (colour) M.smid = ar.upload(smid, st);
  M.col = ar.upload(col, st);
  M.val64 = ar.upload(val, st);
  M.val32 = ar.upload(val32, st);
  if (square) {
    std::vector<double> inv(n);
    std::vector<float> s32(n), dh32(n);
    for (int64_t r = 0; r < n; ++r) {
      inv[r] = 1.0 / ad[r];
      s32[r] = (float)ad[r];
      dh32[r] = (float)(dv[r] / ad[r]);
    }
    M.d64 = ar.upload(dv, st);
    M.i64 = ar.upload(inv, st);
    M.s32 = ar.upload(s32, st);
    M.dh32 = ar.upload(dh32, st);
  }
  return M;
}

// One entry of a row packed by pack_rows (col2: see Sell)
struct RowEntry {
  int32_t col, col2;
  double v;
  float v32;
};

// Row data of pack_rows (empty vectors: not stored): deficit and diagonal
struct RowData {
  std::vector<double> d, diag;
};

// Rows given one by one -> SELL-64 (device): row(i, out) appends row i's
// entries, all of them in the lower part (smid at the slice's end); padding
// entries have value 0 and column pad(i).
template <class F, class G>
Sell pack_rows(Arena &ar, hipStream_t st, int64_t n, bool pairs, F &&row, G &&pad, const RowData &data = RowData()) {
  const int64_t ns = (n + kWave - 1) / kWave;
  std::vector<int64_t> sptr(ns + 1, 0);
  by_slices(ns, 8 * n, [&](int64_t s) {
    std::vector<RowEntry> out;
    for (int64_t i = s * kWave; i < std::min(n, (s + 1) * kWave); ++i) {
      out.clear();
      row(i, out);
      sptr[s + 1] = std::max(sptr[s + 1], (int64_t)out.size() * kWave);
    }
  });
  for (int64_t s = 0; s < ns; ++s) sptr[s + 1] += sptr[s];
  if (ar.count_only) {
    ar.alloc<int64_t>(ns + 1);
    return count_sell(ar, n, sptr[ns], pairs, !data.diag.empty());
  }
  std::vector<int32_t> col(sptr[ns], 0), col2(pairs ? sptr[ns] : 0, -1);
  std::vector<double> val(sptr[ns], 0.0);
  std::vector<float> val32(sptr[ns], 0.0f);
  by_slices(ns, 8 * n, [&](int64_t s) {
    std::vector<RowEntry> out;
    for (int t = 0; t < kWave && s * kWave + t < n; ++t) {
      const int64_t i = s * kWave + t;
      out.clear();
      row(i, out);
      int64_t pos = sptr[s] + t;
      for (const RowEntry &e : out) {
        col[pos] = e.col;
        if (pairs) col2[pos] = e.col2;
        val[pos] = e.v;
        val32[pos] = e.v32;
        pos += kWave;
      }
      for (; pos < sptr[s + 1]; pos += kWave) col[pos] = pad(i);
    }
  });
  Sell M;
  M.nrows = n;
  M.sptr = ar.upload(sptr, st);
  M.smid = M.sptr + 1;
  M.col = ar.upload(col, st);
  if (pairs) M.col2 = ar.upload(col2, st);
  M.val64 = ar.upload(val, st);
  M.val32 = ar.upload(val32, st);
  if (!data.diag.empty()) {
    std::vector<double> inv(n);
    std::vector<float> s32(n), dh32(n);
    for (int64_t i = 0; i < n; ++i) {
      inv[i] = 1.0 / data.diag[i];
      s32[i] = (float)data.diag[i];
      dh32[i] = (float)(data.d[i] / data.diag[i]);
    }
    M.d64 = ar.upload(data.d, st);
    M.i64 = ar.upload(inv, st);
    M.s32 = ar.upload(s32, st);
    M.dh32 = ar.upload(dh32, st);
  }
  return M;
}

// CSR (host) -> CsrG (device).  Square matrices keep only off-diagonals
// (FP64 values; FP32 values a_ij / a_ii with s32 = a_ii).
// G = smallest power of two >= a sixth of the mean row length, clamped to
// [2, 16]: a group of lanes keeps four to eight entries in flight.
// With colkey (rectangular operators gathering from the fine level: the
// spatial rank of column c is (*colkey)[c + coloff]) the rows are stored in
// the order of their smallest column rank and orow maps them back, so that
// the rows one XCD works on gather from one region of the fine vector; each
// row keeps its entries and their order.
// colmap (optional): the stored column of column c is (*colmap)[c].
// zero (optional): the entries of the columns c with (*zero)[c + coloff] != 0
// are left out (the operator's input is zero there).
// like (optional): the same operator packed before with another colmap, whose
// other arrays serve this one too.
CsrG pack_csrg(Arena &ar, hipStream_t st, const Csr &A, bool square, int64_t *stored = nullptr,
               const std::vector<int64_t> *colkey = nullptr, int64_t coloff = 0,
               const std::vector<int32_t> *colmap = nullptr, const std::vector<uint8_t> *zero = nullptr,
               const CsrG *like = nullptr) {
  if (ar.count_only) {
    int64_t nnz = 0;
    for (int64_t r = 0; r < A.nrows; ++r)
      for (int64_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k)
        nnz += !(square && A.idx[k] == r) && !(zero && (*zero)[A.idx[k] + coloff]);
    if (stored) *stored = nnz;
    ar.alloc<int32_t>(nnz);
    CsrG M;
    M.nrows = A.nrows;
    if (like) return M;
    ar.alloc<int32_t>(A.nrows + 1);
    ar.alloc<double>(nnz);
    ar.alloc<float>(nnz);
    if (colkey && !square) ar.alloc<int32_t>(A.nrows);
    if (square) {
      ar.alloc<float>(A.nrows);
      ar.alloc<int32_t>(A.nrows);
    }
    return M;
  }
  std::vector<int32_t> ptr(A.nrows + 1, 0), upper(square ? A.nrows : 0), col;
  std::vector<double> val, d(square ? A.nrows : 0, 0.0);
  std::vector<float> val32;
  col.reserve(A.nnz());
  val.reserve(A.nnz());
  for (int64_t r = 0; r < A.nrows && square; ++r)
    for (int64_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k)
      if (A.idx[k] == r) d[r] = A.val[k];
  std::vector<int64_t> rows(A.nrows);
  std::iota(rows.begin(), rows.end(), 0);
  const bool permute = colkey != nullptr && !square;
  if (permute) {
    std::vector<int64_t> key(A.nrows, INT64_MAX);
    for (int64_t r = 0; r < A.nrows; ++r)
      for (int64_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) key[r] = std::min(key[r], (*colkey)[A.idx[k] + coloff]);
    std::stable_sort(rows.begin(), rows.end(), [&](int64_t a, int64_t b) { return key[a] < key[b]; });
  }
  for (int64_t i = 0; i < A.nrows; ++i) {
    const int64_t r = rows[i];
    for (int64_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
      if (square && A.idx[k] == r) continue;
      if (zero && (*zero)[A.idx[k] + coloff]) continue;
      if (square && A.idx[k] < r) upper[i] = (int32_t)col.size() + 1;
      col.push_back(colmap ? (*colmap)[A.idx[k]] : A.idx[k]);
      val.push_back(A.val[k]);
      val32.push_back(square ? (float)(A.val[k] / d[r]) : (float)A.val[k]);
    }
    ptr[i + 1] = (int32_t)col.size();
    if (square && upper[i] < ptr[i]) upper[i] = ptr[i];  // no earlier column
  }
  double mean = A.nrows ? (double)col.size() / (double)A.nrows : 0.0;
  int G = 2;
  while (G < 16 && G < mean / 6.0) G *= 2;
  if (stored) *stored = (int64_t)col.size();
  CsrG M;
  if (like) {
    M = *like;
    M.col = ar.upload(col, st);
    return M;
  }
  M.nrows = A.nrows;
  M.G = G;
  M.col = ar.upload(col, st);
  M.ptr = ar.upload(ptr, st);
  M.val64 = ar.upload(val, st);
  M.val32 = ar.upload(val32, st);
  if (permute) {
    std::vector<int32_t> orow(rows.begin(), rows.end());
    M.orow = ar.upload(orow, st);
  }
  if (square) {
    std::vector<float> s32(A.nrows);
    for (int64_t r = 0; r < A.nrows; ++r) s32[r] = (float)d[r];
    M.s32 = ar.upload(s32, st);
    M.upper = ar.upload(upper, st);
  }
  return M;
}

// per-precision work vectors, each [n][kMaxBatch]
template <class T>
struct Work {
  T *x = nullptr, *r = nullptr, *z = nullptr, *p = nullptr, *q = nullptr, *w = nullptr, *res = nullptr,
    *resA = nullptr, *tmp = nullptr;
  // FP64 only: the solution as the unevaluated sum xs + xl, into which each
  // restart's correction x is folded
  T *xs = nullptr, *xl = nullptr;
};

struct DLevel {
  Sell As;                      // fine A_bar level: rows [row0, row0 + n) of the fine SELL matrix
  CsrG Ac;                      // coarse levels: standard form
  PatchSweep ps;                // coarse levels: the patches of the sweeps
  int64_t np = 0;               // number of patches
  unsigned long long *begun = nullptr;  // progress of the sweeps (PatchJob)
  unsigned *ended = nullptr;
  bool fine = false;
  int64_t n = 0, row0 = 0;
  int64_t n_top = 0;            // fine levels: rows of the top block in the fine matrix
  std::vector<int64_t> cstart;  // colour ranges, global row indices
  std::vector<int64_t> cstart_top;  // fine level of the whole A_UU: top-block range of each colour
  const SliceRef *order = nullptr;  // fine levels: slice visit order of the residual product
  CsrG P, Pt;                   // prolongation (n x n_next) and restriction
  Sell Ps;                      // fine levels: the prolongation in SELL-64 (a few entries a row)
  double *Cinv = nullptr;       // coarsest level only: its explicit inverse
  double *dpart = nullptr;      // and the dense product's partial sums (dense_chunks(n) x n x kMaxBatch)
  bool coarsest = false;
  // vectors indexed by global row, [n][kMaxBatch], per precision
  double *x64 = nullptr, *g64 = nullptr, *r64 = nullptr;
  float *x32 = nullptr, *g32 = nullptr, *r32 = nullptr;
  template <class T>
  T *&x() {
    if constexpr (std::is_same<T, double>::value) return x64; else return x32;
  }
  template <class T>
  T *&g() {
    if constexpr (std::is_same<T, double>::value) return g64; else return g32;
  }
  template <class T>
  T *&r() {
    if constexpr (std::is_same<T, double>::value) return r64; else return r32;
  }
};

// pinned copies of device results that the host polls
struct HostBox {
  Scal scal;
  double sums[kMaxBatch];
};

// kGraphFP32Reliable: an FP32 iteration followed by the reliable update of
// the mixed-precision solve (the last iteration of every chunk)
enum GraphKind { kGraphFP64 = 0, kGraphFP32 = 1, kGraphMixedPC = 2, kGraphFP32Reliable = 3 };

// the captured graph of one or more PCG iterations
struct IterGraph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

}  // namespace
}  // namespace vemg

struct vemg_solver_s {
  vemg_options opt;
  int device = -1;
  hipStream_t user = nullptr, work = nullptr;
  bool own_stream = true;   // false: work belongs to a server's stream pool
  size_t footprint = 0;     // device bytes of the uploaded setup (counted before the upload)
  hipEvent_t ev = nullptr;
  std::string err;
  bool ready = false;
  vemg::Problem P;
  vemg::Arena ar;
  vemg::Sell A;                           // fine A_UU, difference form
  vemg::Sell E;
  vemg::CsrG Et, Et_res;                  // Et_res: for residuals after a forward sweep (zero_res left out)
  // fine rows without a neighbour of a later colour, whose residual after the
  // forward sweep is zero: a quarter of the entries of the restrictions
  std::vector<uint8_t> zero_res;
  std::vector<vemg::DLevel> S, Ab, SA;  // SA: baseline hierarchy of the whole A_UU (may be empty)
  vemg::Work<double> v64;
  vemg::Work<float> v32;
  double *b = nullptr, *diag = nullptr, *scale_in = nullptr, *scale_out = nullptr, *dscal = nullptr;
  double *part_pq = nullptr, *part_rr = nullptr, *part_rz = nullptr, *part_b = nullptr, *part_t = nullptr, *part_c = nullptr;
  int64_t dot_rows = 0;  // most rows of partial sums of an iteration's dots
  bool sweep_dot = false;  // the backward sweeps form r . z
  int64_t *perm = nullptr;
  int32_t *pos = nullptr;  // natural node -> storage row, -1: fixed
  // slice visit orders (spatial, across colours) of the products over all
  // rows and over the non-top rows
  vemg::SliceRef *order_all = nullptr, *order_bar = nullptr;
  // VL + additive smoother: both cycles in one pair of fine sweeps (unless
  // A_bar's hierarchy is a single dense level); D's rows of colour c are
  // [dstart[c], dstart[c+1]), and merged_Pt restricts the smoother's residual
  // from the extended vector
  bool merged = false;
  vemg::MergedRows M;
  std::vector<int64_t> dstart;
  vemg::CsrG merged_Pt;
  // the top block of the additive smoother's x (rows [0, n_top) of w) is zero
  // for rows of up to w_clean bytes
  int w_clean = vemg::kMaxBatch * (int)sizeof(double);
  vemg::HostBox *host = nullptr;
  vemg::Scal *scal = nullptr;  // two records: between iterations, and within one (launch_pcg_xr)
  int64_t nnz_A = 0, nnz_E = 0;
  std::map<int, vemg::IterGraph> graphs;  // by kind, K and number of iterations
  // false for server lanes once the scheduler runs: a capture on one thread
  // must not coincide with device-wide synchronisation on another
  bool allow_capture = true;
};

namespace vemg {
namespace {

using Handle = vemg_solver_s;

template <class T>
Work<T> &work_of(Handle *h) {
  if constexpr (std::is_same<T, double>::value) return h->v64; else return h->v32;
}

// The patch arrays of a coarse level for its sweeps (PatchSweep): row ranges
// of the stored patches, every row's entry ranges (positions in the level's
// CsrG, which drops the diagonals) and, per patch, F = (D_p + L_p)^{-1} of its
// diagonal block in stored order (forward substitution on the host in FP64)
// and F^T for the backward sweep, both also times D_p rounded to FP32 for the
// row-scaled FP32 operator, in tiles.
void pack_patches(Arena &ar, hipStream_t st, const Level &L, DLevel &dl) {
  static_assert(kPatchRows == kPatchLdsRows, "the patch size of the order and of the sweep kernel differ");
  constexpr int64_t W = kPatchTile, S = kPatchLdsRows + 1;
  const int64_t n = L.n(), np = (int64_t)L.patch_list.size();
  if (n > INT32_MAX) throw DeviceError(VEMG_ERR_DEVICE, "coarse level above 2^31 rows");
  std::vector<PatchDesc> desc(np);
  std::vector<PatchRow> rows(np * S, PatchRow{0, 0, 0, 0});
  std::vector<int32_t> halo, lcol;
  int64_t tiles = 0;
  std::vector<int32_t> patch_of(n), nbr;  // stored patch of each row
  for (int64_t p = 0; p < np; ++p)
    std::fill(patch_of.begin() + L.patch_row[p], patch_of.begin() + L.patch_row[p + 1], (int32_t)p);
  for (int64_t p = 0; p < np; ++p) {
    const int64_t m = L.patch_row[p + 1] - L.patch_row[p], nt = (m + W - 1) / W;
    if (n * kMaxBatch * 8 > UINT32_MAX) throw DeviceError(VEMG_ERR_DEVICE, "coarse level above the sweep kernel's 32-bit offsets");
    if (m > kPatchLdsRows) throw DeviceError(VEMG_ERR_DEVICE, "a patch exceeds the sweep kernel's rows");
    desc[p] = PatchDesc{(int32_t)L.patch_row[p], (int32_t)m, tiles * W * W, (int32_t)halo.size(), 0, 0,
                        (int32_t)nbr.size(), 0, 0};
    // the halo: the listed part of the other patches' rows, ascending
    const int64_t ps = L.patch_row[p], pe = ps + m;
    std::vector<int32_t> out;
    for (int64_t k = L.A.ptr[ps]; k < L.A.ptr[pe]; ++k)
      if (L.A.idx[k] < ps || L.A.idx[k] >= pe) out.push_back(L.A.idx[k]);
    std::sort(out.begin(), out.end());
    out.erase(std::unique(out.begin(), out.end()), out.end());
    for (int32_t j : out)  // ascending rows, so ascending patches
      if ((int32_t)nbr.size() == desc[p].nbr || nbr.back() != patch_of[j]) {
        nbr.push_back(patch_of[j]);
        ++desc[p].nbr_all;
        desc[p].nbr_early += j < ps;
      }
    if ((int64_t)out.size() > kPatchHalo) out.resize(kPatchHalo);
    desc[p].nhalo = (int32_t)out.size();
    for (int32_t j : out) desc[p].nearly += j < ps;
    for (int64_t i = ps; i < pe; ++i)
      for (int64_t k = L.A.ptr[i]; k < L.A.ptr[i + 1]; ++k) {
        const int32_t j = L.A.idx[k];
        if (j == i) continue;
        const auto at = std::lower_bound(out.begin(), out.end(), j);
        lcol.push_back(j >= ps && j < pe ? (int32_t)(j - ps)
                       : at != out.end() && *at == j ? (int32_t)(kPatchLdsRows + (at - out.begin())) : ~j);
      }
    halo.insert(halo.end(), out.begin(), out.end());
    tiles += nt * (nt + 1) / 2;
  }
  std::vector<double> tf, tb;
  std::vector<float> tf32, tb32;
  if (!ar.count_only) {
    tf.assign(tiles * W * W, 0.0);
    tb.assign(tiles * W * W, 0.0);
    tf32.assign(tiles * W * W, 0.0f);
    tb32.assign(tiles * W * W, 0.0f);
    std::vector<double> M, F;
    int64_t diag = 0;  // diagonal entries passed so far: not stored in the CsrG
    for (int64_t p = 0; p < np; ++p) {
      const int64_t ps = L.patch_row[p], m = L.patch_row[p + 1] - ps, pe = ps + m, nt = (m + W - 1) / W;
      M.assign(m * m, 0.0);
      F.assign(m * m, 0.0);
      for (int64_t r = 0; r < m; ++r) {
        const int64_t i = ps + r;
        int32_t at[4];  // entries with columns before the patch, before the row, up to the row, in the patch
        const int64_t lim[4] = {ps, i, i + 1, pe};
        for (int q = 0; q < 4; ++q)
          at[q] = (int32_t)(std::lower_bound(L.A.idx.begin() + L.A.ptr[i], L.A.idx.begin() + L.A.ptr[i + 1],
                                             (int32_t)lim[q]) - L.A.idx.begin());
        const int32_t b = (int32_t)(L.A.ptr[i] - diag), e = (int32_t)(L.A.ptr[i + 1] - diag);
        const int32_t own = (int32_t)(at[0] - diag), late = (int32_t)(at[1] - diag), has = at[2] - at[1];
        rows[p * S + r] = PatchRow{b, own, late, (int32_t)(at[3] - diag - has)};
        rows[p * S + r + 1].b = e - has;
        diag += has;
        for (int64_t k = L.A.ptr[i]; k < L.A.ptr[i + 1]; ++k) {
          const int64_t c = L.A.idx[k] - ps;
          if (c >= 0 && c <= r) M[r * m + c] = L.A.val[k];
        }
      }
      // columns of F = (D + L)^{-1}: forward substitution on unit vectors
      for (int64_t c = 0; c < m; ++c) {
        F[c * m + c] = 1.0 / M[c * m + c];
        for (int64_t r = c + 1; r < m; ++r) {
          double t = 0.0;
          for (int64_t k = c; k < r; ++k) t += M[r * m + k] * F[k * m + c];
          F[r * m + c] = -t / M[r * m + r];
        }
      }
      // entry (r, c) of a tile row that starts at tile t0 with tile column j0
      auto at = [&](int64_t t0, int64_t j0, int64_t r, int64_t c) {
        return desc[p].toff + (t0 + c / W - j0) * W * W + c % W / 4 * 64 + c % 4 * W + r % W;
      };
      for (int64_t r = 0; r < m; ++r) {
        const int64_t I = r / W, f0 = I * (I + 1) / 2, b0 = I * nt - I * (I - 1) / 2;
        for (int64_t c = 0; c <= r; ++c) {
          tf[at(f0, 0, r, c)] = F[r * m + c];
          tf32[at(f0, 0, r, c)] = (float)(F[r * m + c] * M[c * m + c]);
        }
        for (int64_t c = r; c < m; ++c) {
          tb[at(b0, I, r, c)] = F[c * m + r];
          tb32[at(b0, I, r, c)] = (float)(F[c * m + r] * M[c * m + c]);
        }
      }
    }
  }
  dl.ps.desc = ar.upload(desc, st);
  dl.ps.rows = ar.upload(rows, st);
  if (ar.count_only) {
    for (int k = 0; k < 2; ++k) ar.alloc<double>(tiles * W * W);
    for (int k = 0; k < 2; ++k) ar.alloc<float>(tiles * W * W);
  } else {
    dl.ps.tf64 = ar.upload(tf, st);
    dl.ps.tb64 = ar.upload(tb, st);
    dl.ps.tf32 = ar.upload(tf32, st);
    dl.ps.tb32 = ar.upload(tb32, st);
  }
  dl.ps.halo = ar.upload(halo, st);
  dl.ps.lcol = ar.upload(lcol, st);
  dl.ps.nbr = ar.upload(nbr, st);
  dl.np = np;
  dl.begun = ar.alloc<unsigned long long>(1);
  dl.ended = ar.alloc<unsigned>(np);
  if (!ar.count_only) {
    launch_fill<float>(st, (float *)dl.begun, 2, 0.0f, nullptr);
    launch_fill<float>(st, (float *)dl.ended, np, 0.0f, nullptr);
  }
}

enum LevelsOf { kLevelsS = 0, kLevelsAbar = 1, kLevelsSA = 2 };

// fine_Pt: the finest level's restriction where the caller has it
void build_levels(Handle *h, std::vector<Level> &H, std::vector<DLevel> &D, int of, const Csr *fine_Pt = nullptr) {
  hipStream_t st = h->work;
  D.clear();
  for (size_t l = 0; l < H.size(); ++l) {
    Level &L = H[l];
    DLevel dl;
    dl.n = L.n();
    dl.coarsest = (l + 1 == H.size());
    if (of != kLevelsS && l == 0) {
      // fine level: rows of the fine SELL matrix (non-top rows for A_bar,
      // all rows for the whole A_UU), colour ranges in global rows
      dl.fine = true;
      dl.n_top = h->P.n_top;
      dl.As = h->A;
      dl.row0 = of == kLevelsAbar ? h->P.n_top : 0;
      dl.order = of == kLevelsAbar ? h->order_bar : h->order_all;
      dl.cstart = h->P.bar_colour_start;
      if (of == kLevelsSA) {
        const int nc = std::max((int)h->P.top_colour_start.size(), (int)h->P.bar_colour_start.size()) - 1;
        dl.cstart_top = h->P.top_colour_start;
        dl.cstart_top.resize(nc + 1, dl.cstart_top.back());
        dl.cstart.resize(nc + 1, dl.cstart.back());
      }
      dl.x64 = h->v64.w;
      dl.g64 = h->v64.r;
      dl.r64 = h->v64.resA;
      dl.x32 = h->v32.w;
      dl.g32 = h->v32.r;
      dl.r32 = h->v32.resA;
    } else {
      size_t cnt = (size_t)dl.n * kMaxBatch;
      dl.x64 = h->ar.alloc<double>(cnt);
      dl.g64 = h->ar.alloc<double>(cnt);
      dl.x32 = h->ar.alloc<float>(cnt);
      dl.g32 = h->ar.alloc<float>(cnt);
      if (!dl.coarsest) {  // the coarsest is solved by its inverse alone
        dl.Ac = pack_csrg(h->ar, st, L.A, true);
        pack_patches(h->ar, st, L, dl);
        dl.r64 = h->ar.alloc<double>(cnt);
        dl.r32 = h->ar.alloc<float>(cnt);
      }
    }
    if (!dl.coarsest) {
      if (dl.fine)
        dl.Ps = pack_sell(h->ar, st, L.P, false, nullptr, nullptr);
      else
        dl.P = pack_csrg(h->ar, st, L.P, false);
      // the fine level's restriction gathers from fine rows row0 + c
      dl.Pt = dl.fine ? pack_csrg(h->ar, st, fine_Pt ? *fine_Pt : transpose(L.P), false, nullptr, &h->P.loc_rank,
                                  dl.row0, nullptr, &h->zero_res,
                                  of == kLevelsAbar && h->merged ? &h->merged_Pt : nullptr)
                      : pack_csrg(h->ar, st, transpose(L.P), false);
    } else {
      dl.Cinv = h->ar.upload(L.Cinv, st);
      dl.dpart = h->ar.alloc<double>((size_t)dense_chunks(dl.n) * dl.n * kMaxBatch);
    }
    D.push_back(dl);
  }
}

// The coarse part of one or two hierarchies, from levels l[i] (a coarse level,
// or one that is the coarsest) down and up again; a null hierarchy is left
// out.  The two are independent, so levels at the same height above their
// coarsest share their launches, step by step.
template <class T>
struct Cycle {
  std::vector<DLevel> *H = nullptr;
  size_t l = 0;
  int64_t left() const { return H ? (int64_t)(H->size() - l) : 0; }
  DLevel &level() const { return (*H)[l]; }
};

template <class T>
void coarse_cycles(hipStream_t st, int K, Cycle<T> a, Cycle<T> b, const int *done) {
  const int64_t ra = a.left(), rb = b.left();
  if (ra == 0 && rb == 0) return;
  DLevel *L[2];
  int nl = 0;
  if (ra >= rb) L[nl++] = &a.level();
  if (rb >= ra) L[nl++] = &b.level();
  if (L[0]->coarsest) {
    DenseJob<T> J[2];
    for (int i = 0; i < nl; ++i) {
      const int64_t o = L[i]->row0 * K;
      J[i].C = L[i]->Cinv;
      J[i].m = L[i]->n;
      J[i].g = L[i]->template g<T>() + o;
      J[i].x = L[i]->template x<T>() + o;
      J[i].part = L[i]->dpart;
    }
    launch_dense<T>(st, K, J, nl, done);
    return;
  }
  PatchJob<T> gs[2];
  for (int i = 0; i < nl; ++i)
    gs[i] = PatchJob<T>{L[i]->Ac, L[i]->ps, L[i]->np, L[i]->template g<T>(), L[i]->template x<T>(), L[i]->begun,
                        L[i]->ended};
  launch_patch_gs<T>(st, K, kPatchFirst, gs, nl, done);
  Cycle<T> na = a, nb = b;
  if (ra >= rb) ++na.l;
  if (rb >= ra) ++nb.l;
  CsrJob<T> res[2], down[2], up[2];
  for (int i = 0; i < nl; ++i) {
    DLevel &C = i == 0 && ra >= rb ? na.level() : nb.level();
    res[i].A = L[i]->Ac;
    res[i].x = L[i]->template x<T>();
    res[i].y = L[i]->template r<T>();
    down[i].A = L[i]->Pt;
    down[i].x = L[i]->template r<T>();
    down[i].y = C.template g<T>();
    up[i].A = L[i]->P;
    up[i].x = C.template x<T>();
    up[i].y = L[i]->template x<T>();
  }
  launch_csr<T>(st, K, kCsrUpper, res, nl, done);
  launch_csr<T>(st, K, kCsrMult, down, nl, done);
  coarse_cycles<T>(st, K, na, nb, done);
  launch_csr<T>(st, K, kCsrAdd, up, nl, done);
  launch_patch_gs<T>(st, K, kPatchBackward, gs, nl, done);
}

template <class T>
Cycle<T> cycle(std::vector<DLevel> &H, size_t l) {
  Cycle<T> c;
  c.H = &H;
  c.l = l;
  return c;
}

// Sweeps of a fine level on its own (A_bar's, whose top columns multiply the
// smoother vector's top part, which is zero; or the baseline's whole A):
// forward from zero with the residual, and backward.
template <class T>
void fine_forward(hipStream_t st, int K, DLevel &L, const int *done) {
  T *x = L.x<T>(), *g = L.g<T>();
  const bool top = !L.cstart_top.empty();
  for (size_t c = 0; c + 1 < L.cstart.size(); ++c)
    launch_gs<T>(st, K, L.As, top ? L.cstart_top[c] : 0, top ? L.cstart_top[c + 1] : 0, L.cstart[c], L.cstart[c + 1],
                 g, x, done, true);
  launch_spmv<T>(st, K, L.As, 1, L.row0, L.row0 + L.n, x, L.r<T>(), nullptr, done, L.order);
}
template <class T>
void fine_backward(hipStream_t st, int K, DLevel &L, const int *done) {
  const bool top = !L.cstart_top.empty();
  for (size_t c = L.cstart.size() - 1; c-- > 0;)
    launch_gs<T>(st, K, L.As, top ? L.cstart_top[c] : 0, top ? L.cstart_top[c + 1] : 0, L.cstart[c], L.cstart[c + 1],
                 L.g<T>(), L.x<T>(), done, false);
}

// One V-cycle of a hierarchy with a fine level, and the coarse part of a
// second, independent one beside it (its own down job, if given, beside the
// fine level's restriction).
template <class T>
void fine_cycle(hipStream_t st, int K, std::vector<DLevel> &H, Cycle<T> other, const CsrJob<T> *other_down,
                const int *done) {
  DLevel &L = H[0];
  CsrJob<T> down[2];
  int nd = 0;
  if (other_down) down[nd++] = *other_down;
  if (L.coarsest) {
    if (nd) launch_csr<T>(st, K, kCsrMult, down, nd, done);
    coarse_cycles<T>(st, K, other, cycle<T>(H, 0), done);
    return;
  }
  fine_forward<T>(st, K, L, done);
  const int64_t o = L.row0 * K;
  down[nd].A = L.Pt;
  down[nd].x = L.r<T>() + o;
  down[nd++].y = H[1].g<T>();
  launch_csr<T>(st, K, kCsrMult, down, nd, done);
  coarse_cycles<T>(st, K, other, cycle<T>(H, 1), done);
  launch_rect<T>(st, K, L.Ps, true, H[1].x<T>(), L.x<T>() + o, done);
  fine_backward<T>(st, K, L, done);
}

// The rows of sweep colour c: the top's and the non-top block's
struct ColourRows {
  int64_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;
};
int fine_colours(const Problem &P) {
  return std::max((int)P.top_colour_start.size(), (int)P.bar_colour_start.size()) - 1;
}
ColourRows colour_rows(const Problem &P, int c) {
  ColourRows r;
  if (c + 1 < (int)P.top_colour_start.size()) {
    r.a0 = P.top_colour_start[c];
    r.a1 = P.top_colour_start[c + 1];
  }
  if (c + 1 < (int)P.bar_colour_start.size()) {
    r.b0 = P.bar_colour_start[c];
    r.b1 = P.bar_colour_start[c + 1];
  }
  return r;
}

// The restriction of r to the surface; residual: of the residual after a
// forward sweep
template <class T>
CsrJob<T> surface_down(Handle *h, const T *r, bool residual) {
  CsrJob<T> J;
  J.A = residual ? h->Et_res : h->Et;
  J.x = r;
  J.y = h->S[0].g<T>();
  return J;
}

// zz = one vertical-lumping multigrid cycle on rr (Section 6, second
// preconditioner): forward multicolour SOR on A from zero, E~ coarse
// correction through one V-cycle on the surface operator, backward SOR; with
// dense, the additive smoother of a single dense level runs beside the surface
// cycle.
// part (may be null): receives the partial sums of rr . zz; returns their rows
template <class T>
int64_t sor_cycle(Handle *h, int K, const T *rr, T *zz, double *part, const int *done, bool dense = false) {
  hipStream_t st = h->work;
  const Problem &P = h->P;
  const int nc = fine_colours(P);
  Work<T> &v = work_of<T>(h);
  // the forward sweep starts from zero: zz needs no fill
  for (int c = 0; c < nc; ++c) {
    const ColourRows q = colour_rows(P, c);
    launch_gs<T>(st, K, h->A, q.a0, q.a1, q.b0, q.b1, rr, zz, done, true);
  }
  Cycle<T> S, B;
  if (P.n_top > 0) {
    launch_spmv<T>(st, K, h->A, 1, 0, P.n, zz, v.res, nullptr, done, h->order_all);
    const CsrJob<T> J = surface_down<T>(h, v.res, true);
    launch_csr<T>(st, K, kCsrMult, &J, 1, done);
    S = cycle<T>(h->S, 0);
  }
  T *saved = h->Ab[0].g<T>();
  if (dense) {
    h->Ab[0].g<T>() = const_cast<T *>(rr);
    B = cycle<T>(h->Ab, 0);
  }
  coarse_cycles<T>(st, K, S, B, done);
  h->Ab[0].g<T>() = saved;
  if (P.n_top > 0) launch_rect<T>(st, K, h->E, true, h->S[0].x<T>(), zz, done);
  int64_t np = 0;
  for (int c = nc - 1; c >= 0; --c) {
    const ColourRows q = colour_rows(P, c);
    np += launch_gs<T>(st, K, h->A, q.a0, q.a1, q.b0, q.b1, rr, zz, done, false, part ? part + np * K : nullptr);
  }
  return np;
}

// The fine parts of the two cycles in one (MergedRows): the forward sweep of
// rr from zero, the backward sweep (part as in sor_cycle) and, between them,
// the prolongation of both coarse corrections; zz has n + nx rows.
template <class T>
int64_t merged_colour(Handle *h, int K, int c, bool first, const T *rr, T *zz, double *part, const int *done) {
  const ColourRows q = colour_rows(h->P, c);
  const bool d = c + 1 < (int)h->dstart.size();
  return launch_gs_merged<T>(h->work, K, h->A, h->M, q.a0, q.a1, q.b0, q.b1, d ? h->dstart[c] : 0,
                             d ? h->dstart[c + 1] : 0, rr, zz, done, first, part);
}
template <class T>
void merged_forward(Handle *h, int K, const T *rr, T *zz, const int *done) {
  for (int c = 0; c < fine_colours(h->P); ++c) merged_colour<T>(h, K, c, true, rr, zz, nullptr, done);
}
template <class T>
int64_t merged_backward(Handle *h, int K, const T *rr, T *zz, double *part, const int *done) {
  int64_t np = 0;
  for (int c = fine_colours(h->P) - 1; c >= 0; --c)
    np += merged_colour<T>(h, K, c, false, rr, zz, part ? part + np * K : nullptr, done);
  return np;
}
template <class T>
void merged_prolong(Handle *h, int K, T *zz, const int *done) {
  const T *ya = h->Ab[1].x<T>();
  launch_prolong_merged<T>(h->work, K, h->M, h->P.n_top > 0 ? h->S[0].x<T>() : ya, ya, zz, done);
}

// zz = VL_SOR(rr) + Z Vcyc_Abar(Z^T rr) with one pair of fine sweeps for both
// cycles.  part as in sor_cycle.
template <class T>
int64_t merged_cycle(Handle *h, int K, const T *rr, T *zz, double *part, const int *done) {
  hipStream_t st = h->work;
  const Problem &P = h->P;
  Work<T> &v = work_of<T>(h);
  merged_forward<T>(h, K, rr, zz, done);
  launch_res_merged<T>(st, K, h->A, h->M, zz, v.res, done, h->order_all);
  CsrJob<T> down[2];
  int nd = 0;
  if (P.n_top > 0) down[nd++] = surface_down<T>(h, v.res, true);
  down[nd].A = h->merged_Pt;
  down[nd].x = v.res;
  down[nd++].y = h->Ab[1].g<T>();
  launch_csr<T>(st, K, kCsrMult, down, nd, done);
  coarse_cycles<T>(st, K, P.n_top > 0 ? cycle<T>(h->S, 0) : Cycle<T>(), cycle<T>(h->Ab, 1), done);
  merged_prolong<T>(h, K, zz, done);
  return merged_backward<T>(h, K, rr, zz, part, done);
}

// w = Z Vcyc_Abar(Z^T rr) (the additive smoother; rows of the top block of w
// stay zero), with the surface cycle of `other` beside it
template <class T>
void additive_smoother(Handle *h, int K, const T *rr, Cycle<T> other, const CsrJob<T> *other_down, const int *done) {
  T *saved = h->Ab[0].g<T>();
  h->Ab[0].g<T>() = const_cast<T *>(rr);
  fine_cycle<T>(h->work, K, h->Ab, other, other_down, done);
  h->Ab[0].g<T>() = saved;
}

// z = M^{-1} rr in precision T; partial sums of rr . z go to part (rows in
// *np) unless it is null.  part holds dot_rows rows, as part_rz alone does: the
// backward sweeps write one per slice and colour, which for few unknowns of
// many colours is more than the other buffers have.  zz: the handle's own z
// vector (the merged cycles extend it).
template <class T>
void precond(Handle *h, int K, const T *rr, T *zz, double *part, int64_t *np, const int *done) {
  hipStream_t st = h->work;
  const Problem &P = h->P;
  int64_t n = P.n;
  Work<T> &v = work_of<T>(h);
  *np = vec_blocks(n);
  switch (h->opt.pc) {
    case VEMG_PC_VL_ADDITIVE:
      if (h->merged) {
        const int64_t rows = merged_cycle<T>(h, K, rr, zz, h->sweep_dot ? part : nullptr, done);
        if (!h->sweep_dot) break;
        *np = rows;
        return;
      }
      sor_cycle<T>(h, K, rr, zz, nullptr, done, true);
      launch_add_dot<T>(st, K, v.w, rr, zz, P.n_top, n, part ? part : h->part_t, done);
      return;
    case VEMG_PC_VL_ADDITIVE_ONLY:
      if (P.n_top > 0) {
        const CsrJob<T> J = surface_down<T>(h, rr, false);
        additive_smoother<T>(h, K, rr, cycle<T>(h->S, 0), &J, done);
        launch_prolong_sum<T>(st, K, h->E, P.n_top, h->S[0].x<T>(), v.w, rr, zz, part ? part : h->part_t,
                              done);
        *np = sell_blocks(0, n);
        return;
      }
      additive_smoother<T>(h, K, rr, Cycle<T>(), nullptr, done);  // empty surface: the smoother alone
      launch_copy<T>(st, v.w, zz, n * K, done);
      break;
    case VEMG_PC_VL_SOR: {
      const int64_t rows = sor_cycle<T>(h, K, rr, zz, h->sweep_dot ? part : nullptr, done);
      if (!h->sweep_dot) break;
      *np = rows;
      return;
    }
    case VEMG_PC_SA: {
      // one V-cycle of the baseline hierarchy, its fine level on rr -> zz
      DLevel &F = h->SA[0];
      T *sx = F.x<T>(), *sg = F.g<T>();
      F.x<T>() = zz;
      F.g<T>() = const_cast<T *>(rr);
      fine_cycle<T>(st, K, h->SA, Cycle<T>(), nullptr, done);
      F.x<T>() = sx;
      F.g<T>() = sg;
      break;
    }
    case VEMG_PC_JACOBI:
      launch_jacobi<T>(st, K, rr, h->diag, zz, n, done);
      break;
    default:
      launch_copy<T>(st, rr, zz, n * K, done);
      break;
  }
  if (part) launch_dot<T>(st, K, rr, zz, n, part, done);
}

// The additive smoother reads the top columns of its x and takes them as
// zero, so the top block of w must be zero.  Vectors are laid out [n][K], and
// both precisions' w is one array: a call with K columns writes the non-top
// rows from n_top K words on, which a later call with wider rows reads as part
// of its top block.  Every call with K columns calls this first.
void batch_layout(Handle *h, int K) {
  const int64_t m = h->P.n_top;
  const int width = K * (int)(h->opt.precision == VEMG_FP64 ? sizeof(double) : sizeof(float));
  if (width > h->w_clean && m > 0) launch_fill<float>(h->work, h->v32.w, m * width / 4, 0.0f, nullptr);
  h->w_clean = width;
}

// zz = M^{-1} rr in FP32 for FP64 CG (columns scaled by scale_in, rr already
// scaled and rounded into v32.tmp), with the partial sums of rr . zz in part_rz
int64_t precond_mixed(Handle *h, int K, const double *rr, double *zz, const int *done) {
  int64_t n = h->P.n, np = 0;
  precond<float>(h, K, h->v32.tmp, h->v32.z, nullptr, &np, done);
  launch_promote_dot(h->work, K, h->v32.z, h->scale_out, rr, zz, n, h->part_rz, done);
  return vec_blocks(n);
}

// Reliable update of the mixed-precision solve (FP32 PCG on A d = b / ||b||):
// the FP32 correction accumulated since the last update is scaled by ||b||,
// folded into the FP64 solution hi + lo without rounding error and cleared;
// the true residual b - A (hi + lo) is evaluated in extended precision
// (v64.res) and, scaled by 1 / ||b||, replaces the FP32 recurrence residual.
// The search directions are kept.  The kernels run whatever the columns'
// state, so that a chunk always ends with every correction folded.
void reliable_update(Handle *h, int K) {
  hipStream_t st = h->work;
  const int64_t n = h->P.n;
  launch_promote(st, K, h->v32.x, h->scale_out, h->v64.x, n, nullptr);
  launch_fold(st, K, (1u << K) - 1u, h->v64.xs, h->v64.xl, h->v64.x, n);
  launch_fill<float>(st, h->v32.x, n * K, 0.0f, nullptr);
  launch_residual_ext(st, K, h->A, h->b, h->v64.xs, h->v64.xl, h->v64.res);
  launch_demote(st, K, h->v64.res, h->scale_in, h->v32.r, n, nullptr);
}

// One PCG iteration in precision T (kind FP64/FP32) or FP64 with an FP32
// preconditioner (kind MixedPC), on one stream.
template <class T>
void pcg_iteration(Handle *h, int K, int kind) {
  hipStream_t st = h->work;
  int64_t n = h->P.n;
  Work<T> &v = work_of<T>(h);
  launch_spmv<T>(st, K, h->A, 0, 0, n, v.p, v.q, h->part_pq, &h->scal->all_done, h->order_all);
  const bool mixed = kind == kGraphMixedPC;
  Scal *in = h->scal, *mid = h->scal + 1;
  // the partial sums of a scalar step, added in parts first where they are many
  auto sums = [&](const double *p, int64_t np, const Scal *s) {
    if (np <= kCompactFrom) return PartialSums{p, np};
    launch_compact(st, K, p, np, h->part_c, &s->all_done);
    return PartialSums{h->part_c, kCompact};
  };
  const bool fold = pcg_folds(h->dot_rows, K);
  const int64_t nv = vec_blocks(n);
  PartialSums pq = sums(h->part_pq, sell_blocks(0, n), in);
  if (!fold) {
    launch_pcg_alpha(st, K, in, mid, pq);
    pq = PartialSums();
  }
  launch_pcg_xr<T>(st, K, in, mid, pq, v.x, v.r, v.p, v.q, n, h->part_rr, mixed ? h->v32.tmp : nullptr, h->scale_in);
  PartialSums rr{h->part_rr, nv};
  if (!fold || n > kFoldConvMax) {
    launch_pcg_conv(st, K, mid, sums(h->part_rr, nv, mid));
    rr = PartialSums();
  }
  const int *done = &mid->all_done;
  if constexpr (std::is_same<T, float>::value)
    if (kind == kGraphFP32Reliable) reliable_update(h, K);
  int64_t np = 0;
  if (mixed) {
    if constexpr (std::is_same<T, double>::value) np = precond_mixed(h, K, v.r, v.z, done);
  } else {
    precond<T>(h, K, v.r, v.z, h->part_rz, &np, done);
  }
  PartialSums rz{h->part_rz, np};
  if (!fold) {
    launch_pcg_beta(st, K, mid, in, sums(h->part_rz, np, mid));
    rz = PartialSums();
  }
  launch_pcg_p<T>(st, K, mid, in, rr, rz, v.p, v.z, n);
}

void destroy_graphs(Handle *h) {
  for (auto &kv : h->graphs) {
    if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
    if (kv.second.graph) (void)hipGraphDestroy(kv.second.graph);
  }
  h->graphs.clear();
}

// A chunk is poll_every iterations or fewer (chunk_for), after which the host
// reads the flags; the FP32 form's last one ends in the reliable update.  Up to
// kGraphIterations of them are one graph: in a chain of dependent kernels, those of a graph of
// 40 nodes (one iteration) took 1.73 us each and of one of 400 nodes 1.55 us,
// launched one by one 2.4 us and more, bound by the host.  A longer chunk
// repeats the graph of one iteration.
constexpr int kGraphIterations = 16;

template <class T>
void chunk_iterations(Handle *h, int K, int kind, int count, bool last) {
  for (int k = 0; k < count; ++k)
    pcg_iteration<T>(h, K, kind == kGraphFP32 && last && k + 1 == count ? kGraphFP32Reliable : kind);
}

template <class T>
void start_phase(Handle *h, int K, int kind);

// graph of `count` iterations for (kind, K) (0: of the start of a phase),
// captured on first use when allowed
template <class T>
const IterGraph *iteration_graph(Handle *h, int K, int kind, int count, bool last) {
  const int key = ((last && kind == kGraphFP32 ? kGraphFP32Reliable : kind) * 16 + K) * 32 + count;
  auto it = h->graphs.find(key);
  if (it != h->graphs.end()) return &it->second;
  if (!h->allow_capture) return nullptr;
  IterGraph ig;
  HIPCHK(hipStreamBeginCapture(h->work, hipStreamCaptureModeThreadLocal));
  if (count)
    chunk_iterations<T>(h, K, kind, count, last);
  else
    start_phase<T>(h, K, kind);
  HIPCHK(hipStreamEndCapture(h->work, &ig.graph));
  HIPCHK(hipGraphInstantiate(&ig.exec, ig.graph, nullptr, nullptr, 0));
  return &h->graphs.emplace(key, ig).first->second;
}

// z = M^{-1} r, rho = r . z and p = z: the start of a phase
template <class T>
void start_phase(Handle *h, int K, int kind) {
  Work<T> &v = work_of<T>(h);
  int64_t np = 0;
  if (kind == kGraphMixedPC) {
    if constexpr (std::is_same<T, double>::value) {
      launch_demote(h->work, K, v.r, h->scale_in, h->v32.tmp, h->P.n, nullptr);
      np = precond_mixed(h, K, v.r, v.z, nullptr);
    }
  } else {
    precond<T>(h, K, v.r, v.z, h->part_rz, &np, nullptr);
  }
  launch_pcg_set_rho(h->work, K, h->scal, h->part_rz, np);
  launch_copy<T>(h->work, v.z, v.p, h->P.n * K, nullptr);
}

template <class T>
void run_start(Handle *h, int K, int kind) {
  const IterGraph *ig = h->opt.use_graphs ? iteration_graph<T>(h, K, kind, 0, true) : nullptr;
  if (ig)
    HIPCHK(hipGraphLaunch(ig->exec, h->work));
  else
    start_phase<T>(h, K, kind);
}

// iterations of the graph that a chunk of poll iterations repeats
int chunk_unit(int poll) { return poll <= kGraphIterations ? poll : 1; }

// poll iterations (by default poll_every, after which the host reads the flags)
template <class T>
void run_chunk(Handle *h, int K, int kind, int poll = 0) {
  if (!poll) poll = std::max(1, h->opt.poll_every);
  const int unit = chunk_unit(poll);
  for (int done = 0; done < poll; done += unit) {
    const bool last = done + unit == poll;
    const IterGraph *ig = h->opt.use_graphs ? iteration_graph<T>(h, K, kind, unit, last) : nullptr;
    if (ig)
      HIPCHK(hipGraphLaunch(ig->exec, h->work));
    else
      chunk_iterations<T>(h, K, kind, unit, last);
  }
}

Scal read_scal(Handle *h) {
  HIPCHK(hipMemcpyAsync(&h->host->scal, h->scal, sizeof(Scal), hipMemcpyDeviceToHost, h->work));
  HIPCHK(hipStreamSynchronize(h->work));
  return h->host->scal;
}

// the smallest of poll_every, its half and its quarter that holds `need` iterations
int chunk_for(const Handle *h, double need) {
  int c = std::max(1, h->opt.poll_every);
  for (int k = 0; k < 2 && c % 2 == 0 && need <= c / 2; ++k) c /= 2;
  return c;
}

// Captures what later chunks and later solves of (kind, K) may replay, so that
// they capture nothing: which lengths a solve takes depends on its residuals.
// Called while the device works on the first chunk, which hides most of it.
template <class T>
void capture_chunks(Handle *h, int K, int kind) {
  if (!h->opt.use_graphs || kind == kGraphFP32) return;  // that form runs whole chunks alone
  const int poll = std::max(1, h->opt.poll_every);
  for (const int c : {chunk_for(h, poll / 4), chunk_for(h, poll / 2)})
    iteration_graph<T>(h, K, kind, chunk_unit(c), true);
}

// Iterates until every column is done.  need: an estimate of the iterations
// to come; later chunks take theirs from each column's residual reduction over
// the chunk before.  Iterations after the last column is done cost an empty
// launch per kernel (35 us at 17 x 17 x 9, where an iteration takes 60).
// The FP32 form always runs whole chunks, which end in its reliable update.
template <class T>
Scal iterate(Handle *h, int K, int kind, double need = INFINITY) {
  Scal last;
  bool have = false;
  while (true) {
    run_chunk<T>(h, K, kind, kind == kGraphFP32 ? 0 : chunk_for(h, need));
    capture_chunks<T>(h, K, kind);
    const Scal hs = read_scal(h);
    if (hs.all_done) return hs;
    need = 0.0;
    for (int k = 0; k < K; ++k) {
      if (hs.done[k]) continue;
      const double goal = hs.tol2[k] * hs.bnorm2[k];
      const int its = have ? hs.iters[k] - last.iters[k] : 0;
      const double rate = its > 0 ? std::log(hs.rr[k] / last.rr[k]) / its : 0.0;
      need = std::max(need, rate < 0.0 && goal > 0.0 ? std::log(goal / hs.rr[k]) / rate : INFINITY);
    }
    last = hs;
    have = true;
  }
}

// true residual res = b - A (xs + xl) of the extended iterate, evaluated in
// extended precision, and its squared column norms (host)
void true_residual(Handle *h, int K, double *rr_host) {
  hipStream_t st = h->work;
  int64_t n = h->P.n;
  launch_residual_ext(st, K, h->A, h->b, h->v64.xs, h->v64.xl, h->v64.res);
  launch_dot<double>(st, K, h->v64.res, h->v64.res, n, h->part_t, nullptr);
  launch_reduce(st, K, h->part_t, vec_blocks(n), h->dscal);
  HIPCHK(hipMemcpyAsync(h->host->sums, h->dscal, K * sizeof(double), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  std::copy(h->host->sums, h->host->sums + K, rr_host);
}

void upload_scales(Handle *h, int K, const double *in, const double *out) {
  HIPCHK(hipMemcpyAsync(h->scale_in, in, K * sizeof(double), hipMemcpyHostToDevice, h->work));
  HIPCHK(hipMemcpyAsync(h->scale_out, out, K * sizeof(double), hipMemcpyHostToDevice, h->work));
  HIPCHK(hipStreamSynchronize(h->work));
}

struct ColResult {
  int iters = 0;
  double rel = 0.0;
  int status = VEMG_OK;
};

// squared column norms of b (host)
void rhs_norms(Handle *h, int K, double *bb) {
  hipStream_t st = h->work;
  int64_t n = h->P.n;
  launch_dot<double>(st, K, h->b, h->b, n, h->part_b, nullptr);
  launch_reduce(st, K, h->part_b, vec_blocks(n), h->dscal);
  HIPCHK(hipMemcpyAsync(h->host->sums, h->dscal, K * sizeof(double), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  std::copy(h->host->sums, h->host->sums + K, bb);
}

// PCG (FP64, or FP64 with FP32 preconditioner) with restarts from the true
// residual; h->b holds K columns (storage order), result in v64.x.
void solve_cg(Handle *h, int K, double rtol, int max_iter, ColResult *res) {
  batch_layout(h, K);
  hipStream_t st = h->work;
  int64_t n = h->P.n;
  Work<double> &v = h->v64;
  bool mixed = h->opt.precision == VEMG_MIXED_PC;
  int kind = mixed ? kGraphMixedPC : kGraphFP64;
  launch_fill<double>(st, v.x, n * K, 0.0, nullptr);
  launch_fill<double>(st, v.xs, n * K, 0.0, nullptr);
  launch_fill<double>(st, v.xl, n * K, 0.0, nullptr);
  launch_copy<double>(st, h->b, v.r, n * K, nullptr);
  launch_dot<double>(st, K, h->b, h->b, n, h->part_b, nullptr);
  launch_pcg_init(st, K, h->scal, h->part_b, vec_blocks(n), rtol, max_iter, mixed ? h->scale_in : nullptr,
                  h->scale_out);
  const unsigned all = (1u << K) - 1u;
  double prev[kMaxBatch], need = INFINITY;
  bool final_[kMaxBatch];
  int restarts = 0;
  for (int k = 0; k < K; ++k) {
    prev[k] = INFINITY;
    final_[k] = false;
  }
  while (true) {
    run_start<double>(h, K, kind);
    Scal hs = iterate<double>(h, K, kind, need);
    const double *bb = hs.bnorm2;
    // columns already final hold x = 0 and are not updated: folding all is exact for them
    launch_fold(st, K, all, v.xs, v.xl, v.x, n);
    double rr[kMaxBatch];
    true_residual(h, K, rr);
    unsigned keep = 0;
    bool any = false;
    need = 0.0;
    for (int k = 0; k < K; ++k) {
      ColResult &c = res[k];
      c.iters = hs.iters[k];
      if (final_[k]) {
        keep |= 1u << k;
        continue;
      }
      if (bb[k] == 0.0) {
        c.rel = 0.0;
        c.status = VEMG_OK;
      } else if (hs.status[k] == -6 || !std::isfinite(bb[k])) {
        c.rel = NAN;
        c.status = VEMG_ERR_BREAKDOWN;
      } else {
        c.rel = std::sqrt(rr[k] / bb[k]);
        if (c.rel <= rtol) c.status = VEMG_OK;
        else if (hs.iters[k] >= max_iter) c.status = VEMG_WARN_MAXITER;
        else if (restarts >= h->opt.max_restarts || c.rel > 0.5 * prev[k]) c.status = VEMG_WARN_FLOOR;
        else {
          prev[k] = c.rel;
          any = true;
          // at the mean rate so far, and one more
          need = std::max(need, 1.0 + hs.iters[k] * std::log(rtol / c.rel) / std::log(rtol));
          continue;  // restart this column
        }
      }
      final_[k] = true;
      keep |= 1u << k;
    }
    if (!any) break;
    ++restarts;
    launch_copy<double>(st, v.res, v.r, n * K, nullptr);
    launch_pcg_resume(st, K, h->scal, keep);
  }
  launch_round(st, v.xs, v.xl, v.x, n * K);
}

// Mixed precision (VEMG_MIXED_IR): FP64 iterative refinement whose inner FP32
// PCG keeps its Krylov space.  The inner PCG (SpMV, transfers, smoothers and
// vectors in FP32 with per-row scaled operators, inner products accumulated
// in FP64, coarsest solves in FP64) runs on A d = b / ||b||; every poll_every
// iterations a reliable update folds its correction into the FP64 solution
// hi + lo and replaces its residual with the true FP64 residual (evaluated in
// extended precision), without restarting the search directions.  A column
// whose recurrence residual meets rtol is confirmed on that true residual
// and, if it is not met, restarted from it (at most max_restarts times, while
// each restart at least halves it).  h->b holds K columns.
void solve_ir(Handle *h, int K, double rtol, int max_iter, ColResult *res) {
  batch_layout(h, K);
  hipStream_t st = h->work;
  int64_t n = h->P.n;
  Work<float> &v = h->v32;
  double bb[kMaxBatch], sin[kMaxBatch], sout[kMaxBatch];
  rhs_norms(h, K, bb);
  for (int k = 0; k < K; ++k) {
    const double nb = std::sqrt(bb[k]);
    const bool ok = nb > 0.0 && std::isfinite(nb);
    sin[k] = ok ? 1.0 / nb : 0.0;
    sout[k] = ok ? nb : 0.0;
  }
  upload_scales(h, K, sin, sout);
  launch_fill<double>(st, h->v64.x, n * K, 0.0, nullptr);
  launch_fill<double>(st, h->v64.xs, n * K, 0.0, nullptr);
  launch_fill<double>(st, h->v64.xl, n * K, 0.0, nullptr);
  launch_fill<float>(st, v.x, n * K, 0.0f, nullptr);
  launch_demote(st, K, h->b, h->scale_in, v.r, n, nullptr);
  // bnorm2 of the scaled system (about 1); a zero b stops its column at once,
  // a non-finite one (scaled to NaN) as a breakdown
  launch_dot<float>(st, K, v.r, v.r, n, h->part_b, nullptr);
  launch_pcg_init(st, K, h->scal, h->part_b, vec_blocks(n), rtol, max_iter);
  double prev[kMaxBatch];
  bool fin[kMaxBatch];
  int restarts = 0;
  for (int k = 0; k < K; ++k) {
    prev[k] = INFINITY;
    fin[k] = false;
    res[k] = ColResult();
  }
  while (true) {
    run_start<float>(h, K, kGraphFP32);
    Scal hs = iterate<float>(h, K, kGraphFP32);
    // the last iteration folded every correction and left b - A (hi + lo) in v64.res
    launch_dot<double>(st, K, h->v64.res, h->v64.res, n, h->part_t, nullptr);
    launch_reduce(st, K, h->part_t, vec_blocks(n), h->dscal);
    double rr[kMaxBatch];
    HIPCHK(hipMemcpyAsync(rr, h->dscal, K * sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    unsigned keep = 0;
    bool any = false;
    for (int k = 0; k < K; ++k) {
      ColResult &c = res[k];
      c.iters = hs.iters[k];
      if (fin[k]) {
        keep |= 1u << k;
        continue;
      }
      if (bb[k] == 0.0) {
        c.rel = 0.0;
        c.status = VEMG_OK;
      } else if (hs.status[k] == -6 || !std::isfinite(bb[k]) || !std::isfinite(rr[k])) {
        c.rel = NAN;
        c.status = VEMG_ERR_BREAKDOWN;
      } else {
        c.rel = std::sqrt(rr[k] / bb[k]);
        if (c.rel <= rtol) c.status = VEMG_OK;
        else if (hs.iters[k] >= max_iter) c.status = VEMG_WARN_MAXITER;
        else if (restarts >= h->opt.max_restarts || c.rel > 0.5 * prev[k]) c.status = VEMG_WARN_FLOOR;
        else {
          prev[k] = c.rel;
          any = true;
          continue;  // restart this column from its true residual (already in v32.r)
        }
      }
      fin[k] = true;
      keep |= 1u << k;
    }
    if (!any) break;
    ++restarts;
    launch_pcg_resume(st, K, h->scal, keep);
  }
  launch_round(st, h->v64.xs, h->v64.xl, h->v64.x, n * K);
}

// The rows of MergedRows (its comment defines D and R) and their packed forms;
// P0t: A_bar's finest restriction.  Returns the number of extended rows.
int64_t merged_rows(Handle *h, const Csr &P0t) {
  const Problem &P = h->P;
  const Csr &O = P.Aoff;
  const int64_t n = P.n, m = P.n_top;
  h->M = MergedRows();
  h->dstart.clear();
  h->merged = P.Abar.size() > 1;
  if (!h->merged) return 0;
  MergedRows &M = h->M;
  auto on = [&](int64_t i, int64_t j) { return j < m ? 0 : P.colour[j] < P.colour[i] ? -1 : 1; };
  std::vector<uint8_t> dirty(n, 0);
  std::vector<int32_t> drow, rrow, xpos(n, -1), rpos;
  const int ncb = (int)P.bar_colour_start.size() - 1;
  h->dstart.assign(1, 0);
  for (int c = 0; c < ncb; ++c) {
    const int64_t i0 = P.bar_colour_start[c], i1 = P.bar_colour_start[c + 1];
    by_slices((i1 - i0 + kWave - 1) / kWave, 8 * (i1 - i0), [&](int64_t s) {
      for (int64_t i = i0 + s * kWave; i < std::min(i1, i0 + (s + 1) * kWave); ++i)
        for (int64_t k = O.ptr[i]; k < O.ptr[i + 1] && !dirty[i]; ++k) {
          const int64_t j = O.idx[k];
          if (P.colour[j] < c && (j < m || dirty[j])) dirty[i] = 1;
        }
    });
    for (int64_t i = i0; i < i1; ++i) {
      if (dirty[i]) {
        xpos[i] = (int32_t)drow.size();
        drow.push_back((int32_t)i);
      }
    }
    h->dstart.push_back((int64_t)drow.size());
  }
  M.n = n;
  M.n_top = m;
  M.nd = M.nx = (int64_t)drow.size();
  std::vector<uint8_t> differs(n, 0);
  by_slices((n + kWave - 1) / kWave, 8 * n, [&](int64_t s) {
    for (int64_t i = std::max(m, s * kWave); i < std::min(n, (s + 1) * kWave); ++i)
      for (int64_t k = O.ptr[i]; k < O.ptr[i + 1] && !differs[i]; ++k) {
        const int64_t j = O.idx[k];
        differs[i] = P.colour[j] > P.colour[i] && (j < m || dirty[j]);
      }
  });
  for (int64_t i = m; i < n; ++i) {
    if (!differs[i]) continue;
    if (xpos[i] < 0) xpos[i] = (int32_t)M.nx++;
    rrow.push_back((int32_t)i);
    rpos.push_back(xpos[i]);
  }
  M.nr = (int64_t)rrow.size();
  if (n + M.nx > INT32_MAX) throw DeviceError(VEMG_ERR_DEVICE, "too many unknowns for 32-bit columns");
  Arena &ar = h->ar;
  hipStream_t st = h->work;
  // column of neighbour j where the smoother's value is meant
  auto fwd_col = [&](int64_t j) { return (int32_t)(dirty[j] ? n + xpos[j] : j); };
  auto ext_col = [&](int64_t j) {
    if (xpos[j] < 0) throw DeviceError(VEMG_ERR_DEVICE, "merged sweeps: a row outside the extended set is read");
    return (int32_t)(n + xpos[j]);
  };
  auto entry = [&](int64_t i, int64_t k, int32_t col, int32_t col2) {
    return RowEntry{col, col2, O.val[k], (float)(O.val[k] / P.diag[i])};
  };
  RowData dd;
  dd.d.resize(M.nd);
  dd.diag.resize(M.nd);
  for (int64_t q = 0; q < M.nd; ++q) {
    const int64_t i = drow[q];
    double d = P.d[i];
    for (int64_t k = O.ptr[i]; k < O.ptr[i + 1]; ++k)
      if (O.idx[k] < m) d -= O.val[k];
    dd.d[q] = d;
    dd.diag[q] = P.diag[i];
  }
  auto dpad = [&](int64_t q) { return (int32_t)(n + q); };
  // row data that another matrix holds
  auto row_data = [](Sell &to, const Sell &from) {
    to.d64 = from.d64;
    to.i64 = from.i64;
    to.s32 = from.s32;
    to.dh32 = from.dh32;
  };
  M.fwd = pack_rows(ar, st, M.nd, false, [&](int64_t q, std::vector<RowEntry> &out) {
    const int64_t i = drow[q];
    for (int64_t k = O.ptr[i]; k < O.ptr[i + 1]; ++k)
      if (on(i, O.idx[k]) < 0) out.push_back(entry(i, k, fwd_col(O.idx[k]), -1));
  }, dpad);
  M.bwd = pack_rows(ar, st, M.nd, false, [&](int64_t q, std::vector<RowEntry> &out) {
    const int64_t i = drow[q];
    for (int64_t k = O.ptr[i]; k < O.ptr[i + 1]; ++k)
      if (on(i, O.idx[k]) != 0) out.push_back(entry(i, k, ext_col(O.idx[k]), -1));
  }, dpad, dd);
  row_data(M.fwd, M.bwd);
  M.res = pack_rows(ar, st, M.nr, false, [&](int64_t q, std::vector<RowEntry> &out) {
    const int64_t i = rrow[q];
    for (int64_t k = O.ptr[i]; k < O.ptr[i + 1]; ++k)
      if (on(i, O.idx[k]) > 0) out.push_back(entry(i, k, fwd_col(O.idx[k]), -1));
  }, [&](int64_t q) { return rrow[q]; });
  std::vector<float> res_scale(M.nr);
  for (int64_t q = 0; q < M.nr; ++q) res_scale[q] = (float)P.diag[rrow[q]];
  M.res.s32 = ar.upload(res_scale, st);
  M.top = pack_rows(ar, st, m, true, [&](int64_t i, std::vector<RowEntry> &out) {
    for (int64_t k = O.ptr[i]; k < O.ptr[i + 1]; ++k)
      out.push_back(entry(i, k, O.idx[k], O.idx[k] < m ? -1 : ext_col(O.idx[k])));
  }, [&](int64_t i) { return (int32_t)i; });
  row_data(M.top, h->A);  // its first rows
  const Csr &P0 = P.Abar[0].P;
  M.prol = pack_rows(ar, st, n, false, [&](int64_t i, std::vector<RowEntry> &out) {
    if (m > 0)
      for (int64_t k = P.E.ptr[i]; k < P.E.ptr[i + 1]; ++k)
        out.push_back({P.E.idx[k], -1, P.E.val[k], (float)P.E.val[k]});
    if (i >= m)
      for (int64_t k = P0.ptr[i - m]; k < P0.ptr[i - m + 1]; ++k)
        out.push_back({(int32_t)(m + P0.idx[k]), -1, P0.val[k], (float)P0.val[k]});
  }, [&](int64_t) { return (int32_t)m; });
  // the smoother's residual: R's extended rows, else the matrix rows
  std::vector<int32_t> map(n - m);
  for (int64_t i = m; i < n; ++i) map[i - m] = (int32_t)i;
  for (int64_t q = 0; q < M.nr; ++q) map[rrow[q] - m] = (int32_t)(n + rpos[q]);
  h->merged_Pt = pack_csrg(ar, st, P0t, false, nullptr, &P.loc_rank, m, &map, &h->zero_res);
  M.drow = ar.upload(drow, st);
  M.rpos = ar.upload(rpos, st);
  M.xpos = ar.upload(xpos, st);
  return M.nx;
}

constexpr int64_t kSweepDotMax = 65536, kSweepDotMin = 1000000;

// Packs the host setup into HBM.  With h->ar.count_only the same sequence
// of allocations is only counted (no device call), which gives the footprint
// of a handle before (or without) its upload.
void upload(Handle *h) {
  hipStream_t st = h->work;
  Problem &P = h->P;
  int64_t n = P.n, m = P.n_top;
  const bool count = h->ar.count_only;
  h->ar.release();
  if (!count) h->ar.reserve(h->footprint);
  SellSpans spans;
  h->A = pack_sell(h->ar, st, P.Aoff, true, &P.d, &P.diag, &h->nnz_A, &P.colour, &spans);
  h->zero_res.assign(n, 1);
  by_slices((n + kWave - 1) / kWave, P.Aoff.nnz(), [&](int64_t s) {
    for (int64_t i = s * kWave; i < std::min(n, (s + 1) * kWave); ++i)
      for (int64_t k = P.Aoff.ptr[i]; k < P.Aoff.ptr[i + 1] && h->zero_res[i]; ++k)
        if (P.colour[P.Aoff.idx[k]] > P.colour[i]) h->zero_res[i] = 0;
  });
  if (m > 0) {
    h->E = pack_sell(h->ar, st, P.E, false, nullptr, nullptr, &h->nnz_E);
    h->Et = pack_csrg(h->ar, st, P.Et, false, nullptr, &P.loc_rank, 0);
    h->Et_res = pack_csrg(h->ar, st, P.Et, false, nullptr, &P.loc_rank, 0, nullptr, &h->zero_res);
  }
  size_t cnt = (size_t)n * kMaxBatch;
  Csr P0t;
  if (P.Abar.size() > 1) P0t = transpose(P.Abar[0].P);
  const size_t ext = (size_t)(n + merged_rows(h, P0t)) * kMaxBatch;
  // Vectors that are never live together share memory (416 bytes a row).
  Work<double> &v = h->v64;
  Work<float> &f = h->v32;
  for (double **p : {&v.x, &v.r, &v.p, &v.q, &v.w, &v.xs, &v.xl}) *p = h->ar.alloc<double>(cnt);
  for (double **p : {&v.z, &v.res}) *p = h->ar.alloc<double>(ext);
  f.r = h->ar.alloc<float>(cnt);
  f.z = h->ar.alloc<float>(ext);
  f.w = (float *)v.w;  // one precision's smoother at a time (batch_layout)
  // q lives from an iteration's product to its x and r.  Beside it: a single
  // operator's input, a served column's solution, and the FP32
  // preconditioner's residual (as long as q: the extended rows are at most n).
  v.tmp = v.q;
  f.res = (float *)v.q;
  // the smoother's cycle alone and the baseline's need no residual of the SOR cycle
  v.resA = v.res;
  f.resA = f.res;
  // the FP32 preconditioner's input in FP64 CG, which has no FP32 r
  f.tmp = f.r;
  // FP32 PCG keeps in FP64 the solution and the true residual alone
  f.x = (float *)v.p;
  f.p = (float *)v.r;
  f.q = (float *)v.z;
  h->b = h->ar.alloc<double>(cnt);
  h->diag = h->ar.upload(P.diag, st);
  h->perm = h->ar.upload(P.perm, st);
  h->pos = h->ar.upload(std::vector<int32_t>(P.pos.begin(), P.pos.end()), st);
  // The products over all rows visit their slices in spatial order across
  // the colours (a slice's key: the spatial rank of its first row in the
  // range), so that the contiguous part of the visit order one XCD takes is
  // one region of every colour, and a row's neighbours, which lie in the
  // other colours, are gathered through the same XCD's L2.
  auto slice_order = [&](int64_t r0, int64_t r1) {
    const int64_t s0 = r0 / kWave, s1 = (r1 + kWave - 1) / kWave;
    std::vector<int32_t> ord(std::max<int64_t>(s1 - s0, 0));
    std::iota(ord.begin(), ord.end(), 0);
    std::stable_sort(ord.begin(), ord.end(), [&](int32_t a, int32_t b) {
      return P.loc_rank[std::max((s0 + a) * kWave, r0)] < P.loc_rank[std::max((s0 + b) * kWave, r0)];
    });
    std::vector<SliceRef> ref(ord.size());
    for (size_t i = 0; i < ord.size(); ++i) {
      const int64_t s = s0 + ord[i];
      ref[i] = SliceRef{s, spans.sptr[s], spans.smid[s], spans.sptr[s + 1]};
    }
    return h->ar.upload(ref, st);
  };
  h->order_all = slice_order(0, n);
  h->order_bar = slice_order(m, n);
  int64_t npmax = (std::max(sell_blocks(0, n), vec_blocks(n)) + 8) * kMaxBatch;
  // A sweep's dot has a row of partial sums per slice and colour (those a
  // boundary cuts count twice), a dot of its own one per 256 rows and a pass
  // over z and r.  The sweep forms it where its rows are few enough to be added
  // by every block for eight columns (launch_pcg_p: n / 64 rows, up to 65,536
  // unknowns), and again where those of a dot of its own are too many even for
  // one (n / 256, from a million), so that no width loses.  Time of an FP64
  // solve with the sweep's against one of its own, on one handle: 2600 to
  // 61,730 unknowns 0.96 to 1.00; 70,698 and 100,819 one column 0.98 to 0.99,
  // eight 1.00 to 1.02; 198,743 and 255,024 0.96 to 0.99; 330,749 to 752,432 one
  // column 1.00 to 1.04, eight 0.97 to 0.98; 1,033,856 0.97 to 0.99.  By the mesh
  // alone, so that a batch's columns keep the single column's sums.
  h->sweep_dot = n <= kSweepDotMax || n >= kSweepDotMin;
  h->dot_rows = h->sweep_dot ? n / kWave + 4 * (fine_colours(P) + 1) : vec_blocks(n);
  h->part_pq = h->ar.alloc<double>(npmax);
  h->part_rr = h->ar.alloc<double>(npmax);
  h->part_rz = h->ar.alloc<double>(std::max(npmax, h->dot_rows * kMaxBatch));
  h->part_c = h->ar.alloc<double>(kCompact * kMaxBatch);
  h->part_b = h->ar.alloc<double>(npmax);
  h->part_t = h->ar.alloc<double>(npmax);
  h->dscal = h->ar.alloc<double>(kMaxBatch);
  h->scale_in = h->ar.alloc<double>(kMaxBatch);
  h->scale_out = h->ar.alloc<double>(kMaxBatch);
  h->scal = h->ar.alloc<Scal>(2);
  if (!count) {
    // every column starts finished (no right-hand side yet)
    launch_fill<double>(st, h->part_b, kMaxBatch, 0.0, nullptr);
    launch_pcg_init(st, kMaxBatch, h->scal, h->part_b, 1, 1.0, 1);
    // the top block of the smoother's vector stays zero
    launch_fill<double>(st, h->v64.w, (int64_t)cnt, 0.0, nullptr);
  }
  if (m > 0) build_levels(h, P.S, h->S, kLevelsS);
  build_levels(h, P.Abar, h->Ab, kLevelsAbar, &P0t);
  h->SA.clear();
  if (!P.SA.empty()) build_levels(h, P.SA, h->SA, kLevelsSA);
  if (!count) HIPCHK(hipStreamSynchronize(st));
}

// device bytes that upload() allocates for the current host setup; the
// handle's device fields are left cleared, so upload() must follow on a
// device handle
size_t count_upload_bytes(Handle *h) {
  Arena saved = std::move(h->ar);
  h->ar = Arena();
  h->ar.count_only = true;
  upload(h);
  size_t b = h->ar.bytes;
  h->ar = std::move(saved);
  return b;
}

void sync_in(Handle *h) {
  HIPCHK(hipEventRecord(h->ev, h->user));
  HIPCHK(hipStreamWaitEvent(h->work, h->ev, 0));
}

// y = A x in natural order; ux, uy: n values each.  On the caller's stream:
// every call leaves the work stream idle, and an event between two queues
// costs more than the product of a small mesh.
void matvec(Handle *h, const double *x, double *y, double *ux, double *uy) {
  const int64_t n = h->P.n, N = h->P.n_nodes;
  launch_gather_batch(h->user, 1, x, N, h->perm, ux, n, 1);
  launch_spmv<double>(h->user, 1, h->A, 0, 0, n, ux, uy, nullptr, nullptr, h->order_all);
  launch_scatter_batch(h->user, 1, uy, h->pos, y, N, 1);
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(h->user));
}

int batch_width(int m) {
  if (m >= 8) return 8;
  if (m >= 4) return 4;
  if (m >= 2) return 2;
  return 1;
}

int do_solve(Handle *h, int nrhs, const double *b_nat, double *x_nat, double rtol, int max_iter, int *iters,
             double *relres) {
  hipStream_t st = h->work;
  int64_t n = h->P.n, N = h->P.n_nodes;
  sync_in(h);
  int worst = VEMG_OK;
  for (int first = 0; first < nrhs;) {
    int m = nrhs - first;
    int K = batch_width(m);
    if (m > 4 && m < 8) K = 8;  // pad small remainders up rather than splitting
    else if (m == 3) K = 4;
    int cols = std::min(K, m);
    launch_gather_batch(st, K, b_nat + (int64_t)first * N, N, h->perm, h->b, n, cols);
    ColResult res[kMaxBatch];
    if (h->opt.precision == VEMG_MIXED_IR)
      solve_ir(h, K, rtol, max_iter, res);
    else
      solve_cg(h, K, rtol, max_iter, res);
    launch_scatter_batch(st, K, h->v64.x, h->pos, x_nat + (int64_t)first * N, N, cols);
    for (int k = 0; k < cols; ++k) {
      if (iters) iters[first + k] = res[k].iters;
      if (relres) relres[first + k] = res[k].rel;
      int s = res[k].status;
      if (s < 0 || (worst >= 0 && s > worst)) worst = s;
    }
    first += cols;
  }
  HIPCHK(hipStreamSynchronize(st));
  return worst;
}

template <class T>
void apply_op(Handle *h, int op, const T *in, T *out) {
  batch_layout(h, 1);
  hipStream_t st = h->work;
  const Problem &P = h->P;
  int64_t n = P.n, m = P.n_top;
  Work<T> &v = work_of<T>(h);
  CsrJob<T> et;
  et.A = h->Et;
  et.x = in;
  et.y = out;
  switch (op) {
    case VEMG_OP_A:
      launch_spmv<T>(st, 1, h->A, 0, 0, n, in, out, nullptr, nullptr, h->order_all);
      break;
    case VEMG_OP_PRECOND: {
      launch_copy<T>(st, in, v.tmp, n, nullptr);
      int64_t np = 0;
      precond<T>(h, 1, v.tmp, v.z, nullptr, &np, nullptr);  // z alone: no partial sums of r . z
      launch_copy<T>(st, v.z, out, n, nullptr);
      break;
    }
    case VEMG_OP_ET:
      launch_csr<T>(st, 1, kCsrMult, &et, 1, nullptr);
      break;
    case VEMG_OP_E:
      launch_rect<T>(st, 1, h->E, false, in, out, nullptr);
      break;
    case VEMG_OP_VCYCLE_S:
      launch_copy<T>(st, in, h->S[0].g<T>(), m, nullptr);
      coarse_cycles<T>(st, 1, cycle<T>(h->S, 0), Cycle<T>(), nullptr);
      launch_copy<T>(st, h->S[0].x<T>(), out, m, nullptr);
      break;
    case VEMG_OP_VCYCLE_ABAR: {
      launch_copy<T>(st, in, v.tmp + m, n - m, nullptr);
      additive_smoother<T>(h, 1, v.tmp, Cycle<T>(), nullptr, nullptr);
      launch_copy<T>(st, v.w + m, out, n - m, nullptr);
      break;
    }
    case VEMG_OP_GS_FWD: {
      for (int c = 0; c < fine_colours(P); ++c) {
        const ColourRows q = colour_rows(P, c);
        launch_gs<T>(st, 1, h->A, q.a0, q.a1, q.b0, q.b1, in, out, nullptr, true);
      }
      break;
    }
  }
}

// The handle's work on the caller's stream while this lives: every call leaves
// the work stream idle, so nothing waits between the two.
struct OnCallersStream {
  Handle *h;
  hipStream_t saved;
  explicit OnCallersStream(Handle *h_) : h(h_), saved(h_->work) { h->work = h->user; }
  ~OnCallersStream() { h->work = saved; }
};

// One application, launched directly on the caller's stream: with an event
// between that and the handle's own (and a clear of the scalars, which no
// operator reads), a preconditioner's application on a small mesh took 117 us,
// without 82 (see matvec).
int do_apply(Handle *h, int op, const double *in, double *out) {
  const Problem &P = h->P;
  int64_t n = P.n, m = P.n_top;
  if (op < VEMG_OP_A || op > VEMG_OP_GS_FWD) return VEMG_ERR_INVALID_ARG;
  if ((op == VEMG_OP_ET || op == VEMG_OP_E || op == VEMG_OP_VCYCLE_S) && m == 0) return VEMG_ERR_STATE;
  int64_t nin = (op == VEMG_OP_E || op == VEMG_OP_VCYCLE_S) ? m : (op == VEMG_OP_VCYCLE_ABAR ? n - m : n);
  int64_t nout = (op == VEMG_OP_ET || op == VEMG_OP_VCYCLE_S) ? m : (op == VEMG_OP_VCYCLE_ABAR ? n - m : n);
  const OnCallersStream here(h);
  hipStream_t st = h->work;
  if (h->opt.precision == VEMG_FP64) {
    apply_op<double>(h, op, in, out);
  } else {
    double one = 1.0, ones[kMaxBatch];
    for (double &o : ones) o = one;
    upload_scales(h, 1, ones, ones);
    float *in32 = h->v32.res, *out32 = h->v32.q;
    launch_demote(st, 1, in, h->scale_in, in32, nin, nullptr);
    apply_op<float>(h, op, in32, out32);
    launch_promote(st, 1, out32, h->scale_out, out, nout, nullptr);
  }
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(st));
  return VEMG_OK;
}

template <class T>
void time_once(Handle *h, int op, int K) {
  hipStream_t st = h->work;
  const Problem &P = h->P;
  int64_t n = P.n;
  Work<T> &v = work_of<T>(h);
  if (op == VEMG_OP_A) {
    launch_spmv<T>(st, K, h->A, 0, 0, n, v.p, v.q, h->part_pq, nullptr, h->order_all);
    return;
  }
  if (op == VEMG_OP_ET) {
    const CsrJob<T> J = surface_down<T>(h, v.r, false);
    launch_csr<T>(st, K, kCsrMult, &J, 1, nullptr);
    return;
  }
  if (op == VEMG_OP_E) {
    launch_rect<T>(st, K, h->E, true, h->S[0].x<T>(), v.z, nullptr);
    return;
  }
  if (op == VEMG_OP_COARSEST) {
    DLevel &L = h->S.back();
    const DenseJob<T> J{L.Cinv, L.n, L.g<T>(), L.x<T>(), L.dpart};
    launch_dense<T>(st, K, &J, 1, nullptr);
    return;
  }
  if (op == VEMG_OP_GS_COARSE) {
    DLevel &L = h->Ab[1];
    const PatchJob<T> J{L.Ac, L.ps, L.np, L.g<T>(), L.x<T>(), L.begun, L.ended};
    launch_patch_gs<T>(st, K, kPatchForward, &J, 1, nullptr);
    return;
  }
  switch (op) {
    case VEMG_OP_MERGED_FWD: merged_forward<T>(h, K, v.r, v.z, nullptr); return;
    case VEMG_OP_MERGED_RES: launch_res_merged<T>(st, K, h->A, h->M, v.z, v.res, nullptr, h->order_all); return;
    case VEMG_OP_MERGED_PROLONG: merged_prolong<T>(h, K, v.z, nullptr); return;
    case VEMG_OP_MERGED_BWD: merged_backward<T>(h, K, v.r, v.z, h->sweep_dot ? h->part_rz : nullptr, nullptr); return;
  }
  for (int c = 0; c < fine_colours(P); ++c) {
    const ColourRows q = colour_rows(P, c);
    launch_gs<T>(st, K, h->A, q.a0, q.a1, q.b0, q.b1, v.r, v.z, nullptr, false);
  }
}

int do_time(Handle *h, int op, int K, int reps, double *avg_ms, int *launches) {
  hipStream_t st = h->work;
  const Problem &P = h->P;
  int64_t n = P.n;
  const bool merged = op >= VEMG_OP_MERGED_FWD && op <= VEMG_OP_MERGED_BWD;
  if (op != VEMG_OP_A && op != VEMG_OP_GS_FWD && op != VEMG_OP_GS_COARSE && op != VEMG_OP_ET && op != VEMG_OP_E &&
      op != VEMG_OP_COARSEST && !merged)
    return VEMG_ERR_INVALID_ARG;
  if (merged && !h->merged) return VEMG_ERR_STATE;
  if (op == VEMG_OP_COARSEST && (P.n_top == 0 || h->S.empty())) return VEMG_ERR_STATE;
  if (op == VEMG_OP_GS_COARSE && (h->Ab.size() < 2 || h->Ab[1].coarsest)) return VEMG_ERR_STATE;
  if ((op == VEMG_OP_ET || op == VEMG_OP_E) && (P.n_top == 0 || h->S.empty())) return VEMG_ERR_STATE;
  if (K != 1 && K != 2 && K != 4 && K != 8) return VEMG_ERR_INVALID_ARG;
  batch_layout(h, K);
  int nc = fine_colours(P);
  if (op == VEMG_OP_GS_COARSE) {
    nc = 1;
    DLevel &L = h->Ab[1];
    if (h->opt.precision == VEMG_MIXED_IR) {
      launch_fill<float>(st, L.g32, L.n * K, 1.0f, nullptr);
      launch_fill<float>(st, L.x32, L.n * K, 0.0f, nullptr);
    } else {
      launch_fill<double>(st, L.g64, L.n * K, 1.0, nullptr);
      launch_fill<double>(st, L.x64, L.n * K, 0.0, nullptr);
    }
  }
  bool f32 = h->opt.precision == VEMG_MIXED_IR;
  if (op == VEMG_OP_E) {
    if (f32)
      launch_fill<float>(st, h->S[0].x32, P.n_top * K, 1.0f, nullptr);
    else
      launch_fill<double>(st, h->S[0].x64, P.n_top * K, 1.0, nullptr);
  }
  if (f32) {
    launch_fill<float>(st, h->v32.p, n * K, 1.0f, nullptr);
    launch_fill<float>(st, h->v32.r, n * K, 1.0f, nullptr);
    launch_fill<float>(st, h->v32.z, (n + h->M.nx) * K, 0.0f, nullptr);
  } else {
    launch_fill<double>(st, h->v64.p, n * K, 1.0, nullptr);
    launch_fill<double>(st, h->v64.r, n * K, 1.0, nullptr);
    launch_fill<double>(st, h->v64.z, (n + h->M.nx) * K, 0.0, nullptr);
  }
  if (op == VEMG_OP_MERGED_PROLONG)
    for (DLevel *L : {P.n_top > 0 ? &h->S[0] : &h->Ab[1], &h->Ab[1]}) {
      launch_fill<float>(st, L->x32, L->n * K, 1.0f, nullptr);
      launch_fill<double>(st, L->x64, L->n * K, 1.0, nullptr);
    }
  auto once = [&]() {
    if (f32) time_once<float>(h, op, K); else time_once<double>(h, op, K);
  };
  once();
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  HIPCHK(hipEventRecord(e0, st));
  for (int k = 0; k < reps; ++k) once();
  HIPCHK(hipEventRecord(e1, st));
  HIPCHK(hipEventSynchronize(e1));
  float ms = 0.0f;
  HIPCHK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *avg_ms = (double)ms / reps;
  if (op == VEMG_OP_COARSEST) {
    DLevel &L = h->S.back();
    if (h->opt.precision == VEMG_MIXED_IR)
      launch_fill<float>(st, L.g32, L.n * K, 1.0f, nullptr);
    else
      launch_fill<double>(st, L.g64, L.n * K, 1.0, nullptr);
    HIPCHK(hipStreamSynchronize(st));
  }
  if (launches) {
    const bool sweep = op == VEMG_OP_GS_FWD || op == VEMG_OP_GS_COARSE || op == VEMG_OP_MERGED_FWD || op == VEMG_OP_MERGED_BWD;
    *launches = sweep ? nc : 1;
  }
  return VEMG_OK;
}

template <class T>
int export_vec(const std::vector<T> &v, void *buf, size_t *bytes) {
  size_t need = v.size() * sizeof(T);
  if (!buf) {
    *bytes = need;
    return VEMG_OK;
  }
  if (*bytes < need) return VEMG_ERR_INVALID_ARG;
  if (need) std::memcpy(buf, v.data(), need);
  *bytes = need;
  return VEMG_OK;
}

int export_csr(const Csr &A, const std::string &what, void *buf, size_t *bytes) {
  if (what == "ptr") return export_vec(A.ptr, buf, bytes);
  if (what == "idx") return export_vec(A.idx, buf, bytes);
  if (what == "val") return export_vec(A.val, buf, bytes);
  return VEMG_ERR_INVALID_ARG;
}

int do_export(Handle *h, const std::string &name, void *buf, size_t *bytes) {
  const Problem &P = h->P;
  if (name == "perm") return export_vec(P.perm, buf, bytes);
  if (name == "colour") return export_vec(P.colour, buf, bytes);
  if (name == "d") return export_vec(P.d, buf, bytes);
  if (name == "diag") return export_vec(P.diag, buf, bytes);
  if (name == "S_perm") return export_vec(P.S_perm, buf, bytes);
  if (name == "graphs") return export_vec(std::vector<int64_t>{(int64_t)h->graphs.size()}, buf, bytes);
  auto dot = name.find('.');
  if (dot == std::string::npos) return VEMG_ERR_INVALID_ARG;
  std::string head = name.substr(0, dot), rest = name.substr(dot + 1);
  if (head == "Aoff") return export_csr(P.Aoff, rest, buf, bytes);
  if (head == "E") return export_csr(P.E, rest, buf, bytes);
  if (head == "S" || head == "Abar" || head == "SA") {
    const std::vector<Level> &H = head == "S" ? P.S : head == "Abar" ? P.Abar : P.SA;
    auto dot2 = rest.find('.');
    if (dot2 == std::string::npos) return VEMG_ERR_INVALID_ARG;
    size_t l = (size_t)std::stoul(rest.substr(0, dot2));
    std::string what = rest.substr(dot2 + 1);
    if (l >= H.size()) return VEMG_ERR_INVALID_ARG;
    const Level &L = H[l];
    if (what.rfind("A.", 0) == 0) return export_csr(L.A, what.substr(2), buf, bytes);
    if (what.rfind("P.", 0) == 0) return export_csr(L.P, what.substr(2), buf, bytes);
    if (what == "colour") return export_vec(L.colour, buf, bytes);
    if (what == "rank") return export_vec(L.rank, buf, bytes);
    if (what == "patch") return export_vec(L.patch, buf, bytes);
    if (what == "pcolour") return export_vec(L.pcolour, buf, bytes);
    if (what == "lcolour") return export_vec(L.lcolour, buf, bytes);
    if (what == "pc_start") return export_vec(L.pc_start, buf, bytes);
    if (what == "patch_row") return export_vec(L.patch_row, buf, bytes);
    if (what == "seg_ptr") return export_vec(L.seg_ptr, buf, bytes);
    if (what == "seg_row") return export_vec(L.seg_row, buf, bytes);
    if (what == "node") return export_vec(L.node, buf, bytes);
    if (what == "agg") return export_vec(L.agg, buf, bytes);
    if (what == "Cinv") return export_vec(L.Cinv, buf, bytes);
  }
  return VEMG_ERR_INVALID_ARG;
}

// A non-blocking stream with a hardware queue of its own: no implicit
// ordering with the legacy null stream (so another thread's work cannot join
// a graph being captured on it; ordering with the caller's stream is
// explicit, see sync_in), and, being created with a CU mask (every CU, so
// nothing is restricted), it does not share its queue, so a solve cannot end
// up serialised behind another stream's work.
hipError_t create_queue_stream(int device, hipStream_t *st) {
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return e;
  std::vector<uint32_t> mask((prop.multiProcessorCount + 31) / 32, 0xffffffffu);
  return hipExtStreamCreateWithCUMask(st, (uint32_t)mask.size(), mask.data());
}

int fail(Handle *h, int code, const std::string &msg) {
  if (h) h->err = msg;
  return code;
}

template <class F>
int guarded(Handle *h, F &&f) {
  // a call that fails leaves nothing running either
  struct Drain {
    Handle *h;
    ~Drain() {
      if (!h || !h->work || !std::uncaught_exceptions()) return;
      (void)hipStreamSynchronize(h->work);
      (void)hipStreamSynchronize(h->user);
    }
  };
  try {
    if (h && h->device >= 0) {
      hipError_t e = hipSetDevice(h->device);
      if (e != hipSuccess) return fail(h, VEMG_ERR_DEVICE, hipGetErrorString(e));
    }
    Drain drain{h};
    return f();
  } catch (const SetupError &e) {
    return fail(h, e.code, e.what());
  } catch (const DeviceError &e) {
    return fail(h, e.code, e.what());
  } catch (const std::bad_alloc &) {
    return fail(h, VEMG_ERR_OOM, "host allocation failed");
  } catch (const std::exception &e) {
    return fail(h, VEMG_ERR_DEVICE, e.what());
  }
}

}  // namespace
}  // namespace vemg


// ============================================================== static buffer
// Device memory for vemg_matvec_noalloc, which allocates nothing: a
// file-scope array that every GPU the library runs on holds until the process
// ends.  In host code its name is only a stand-in; the device address on each
// GPU comes from hipGetSymbolAddress, looked up once per device.
namespace vemg {

constexpr int64_t kScratchRows = int64_t(1) << 21;  // unknowns: two vectors of this length, 32 MiB

namespace {

__device__ __align__(256) double scratch[2 * kScratchRows];

std::mutex scratch_mu;
std::map<int, double *> scratch_addr;  // device ordinal -> address of scratch on that device

// address of the static buffer on `device` (the current device)
double *scratch_of(int device) {
  std::lock_guard<std::mutex> lk(scratch_mu);
  auto it = scratch_addr.find(device);
  if (it != scratch_addr.end()) return it->second;
  void *p = nullptr;
  HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
  scratch_addr[device] = (double *)p;
  return (double *)p;
}

}  // namespace
}  // namespace vemg

// ============================================================== serving
namespace vemg {
namespace {

double now_s() {
  using namespace std::chrono;
  return duration<double>(steady_clock::now().time_since_epoch()).count();
}

// One solve request.  The submitting thread fills it under the server lock;
// afterwards the scheduler thread owns iters, rel, status and cols_left
// until it sets done (under the lock), after which only readers remain.
struct SReq {
  uint64_t id = 0;
  int mesh = 0, nrhs = 0, max_iter = 0;
  const double *b = nullptr;
  double *x = nullptr;
  double rtol = 0.0, t_submit = 0.0, t_done = 0.0;
  int cols_left = 0, status = VEMG_OK;
  bool done = false;
  std::vector<int> iters;
  std::vector<double> rel;
};

// A column slot of a lane.  It points at its request directly: requests are
// owned by unique_ptr and never move, so the scheduler reaches them without
// touching the server's request list.
struct SSlot {
  SReq *req = nullptr;
  int col = 0, restarts = 0;
  double prev = INFINITY;
};

struct Lane {
  vemg_solver_s *h = nullptr;
  bool resident = false;
  size_t footprint = 0;
  std::deque<std::pair<SReq *, int>> queue;  // (request, column), scheduler thread only
  SSlot slot[kMaxBatch];
  bool launched = false;
  uint64_t last_used = 0;
  Scal *scal_host = nullptr;  // pinned copy of the lane's scalars after its last chunk
  hipEvent_t scal_ready = nullptr;
  bool busy() const {
    if (!queue.empty()) return true;
    for (auto &s : slot)
      if (s.req) return true;
    return false;
  }
};

// kServerStreams streams serve every lane (lane i uses stream i mod
// kServerStreams), each created with a (full) CU mask so that it has a
// hardware queue of its own (a process has four).
constexpr int kServerStreams = 4;

}  // namespace
}  // namespace vemg

struct vemg_server_s {
  int device = 0;
  size_t budget = 0;
  vemg_options opt;
  hipStream_t streams[vemg::kServerStreams] = {};
  std::vector<std::unique_ptr<vemg::Lane>> lanes;
  std::vector<std::unique_ptr<vemg::SReq>> reqs;  // owner; appended under mu
  std::map<uint64_t, vemg::SReq *> by_id;
  std::deque<vemg::SReq *> incoming, completed;
  std::mutex mu;
  std::condition_variable cv, cv_done;
  std::thread worker;
  bool stop = false, started = false;
  uint64_t next_id = 1, tick = 0;
  std::string err;
  double first_submit = -1.0, last_done = -1.0;
  // written by the scheduler thread, read by vemg_server_get_stats
  std::atomic<size_t> used{0};
  std::atomic<int64_t> chunks{0}, uploads{0}, evictions{0}, cols_done{0}, active_slots{0};
  int64_t reqs_base = 0;  // requests before the last statistics reset
};

namespace vemg {
namespace {

using Server = vemg_server_s;

void lane_release(Server *sv, Lane &L) {
  destroy_graphs(L.h);
  L.h->ar.release();
  L.resident = false;
  sv->used -= L.footprint;
  sv->evictions++;
}

// make a lane resident, evicting idle lanes (least recently used first)
bool lane_admit(Server *sv, Lane &L) {
  if (L.resident) return true;
  while (sv->budget && sv->used + L.footprint > sv->budget) {
    Lane *victim = nullptr;
    for (auto &o : sv->lanes)
      if (o->resident && !o->busy() && (!victim || o->last_used < victim->last_used)) victim = o.get();
    if (!victim) return false;
    lane_release(sv, *victim);
  }
  upload(L.h);
  if (L.h->ar.bytes != L.footprint)
    throw DeviceError(VEMG_ERR_DEVICE, "device allocations differ from the counted footprint");
  L.resident = true;
  sv->used += L.footprint;
  sv->uploads++;
  return true;
}

// each slot stops on its own request's tolerance and iteration cap
SlotStop lane_stop(const Lane &L) {
  SlotStop st;
  for (int k = 0; k < kMaxBatch; ++k) {
    const SReq *q = L.slot[k].req;
    st.tol[k] = q ? q->rtol : 1.0;
    st.maxit[k] = q ? q->max_iter : 1;
  }
  return st;
}

// (re)start the slot columns in mask: join (x = 0, r = b) or restart (r = res)
void lane_start(Lane &L, unsigned mask, bool restart) {
  Handle *h = L.h;
  batch_layout(h, kMaxBatch);
  hipStream_t st = h->work;
  int64_t n = h->P.n, N = h->P.n_nodes;
  if (!restart)
    for (int k = 0; k < kMaxBatch; ++k)
      if ((mask >> k) & 1u) {
        const SReq &q = *L.slot[k].req;
        launch_gather(st, kMaxBatch, k, q.b + (int64_t)L.slot[k].col * N, h->perm, h->b, n);
      }
  launch_slot_vectors(st, mask, restart, h->b, h->v64.res, h->v64.xs, h->v64.xl, h->v64.x, h->v64.r, n);
  launch_dot<double>(st, kMaxBatch, h->b, h->b, n, h->part_b, nullptr);
  launch_slot_scalars(st, mask, restart, h->scal, h->part_b, vec_blocks(n), lane_stop(L), h->scale_in,
                      h->scale_out);
  int64_t np = 0;
  if (h->opt.precision != VEMG_FP64) {
    launch_demote(st, kMaxBatch, h->v64.r, h->scale_in, h->v32.tmp, n, nullptr);
    np = precond_mixed(h, kMaxBatch, h->v64.r, h->v64.z, nullptr);
  } else
    precond<double>(h, kMaxBatch, h->v64.r, h->v64.z, h->part_rz, &np, nullptr);
  launch_slot_rho(st, mask, h->scal, h->part_rz, np);
  launch_slot_copy(st, mask, h->v64.z, h->v64.p, n);
}

void finish_request(Server *sv, SReq &q) {
  std::lock_guard<std::mutex> lk(sv->mu);
  q.done = true;
  q.t_done = now_s();
  sv->completed.push_back(&q);
  sv->last_done = q.t_done;
  sv->cv_done.notify_all();
}

// columns that finished their chunk: confirm on the FP64 true residual and
// retire them, or restart them from the true residual
void lane_collect(Server *sv, Lane &L) {
  Handle *h = L.h;
  hipStream_t st = h->work;
  HIPCHK(hipEventSynchronize(L.scal_ready));
  const Scal hs = *L.scal_host;
  unsigned fin = 0;
  for (int k = 0; k < kMaxBatch; ++k)
    if (L.slot[k].req && hs.done[k]) fin |= 1u << k;
  if (!fin) return;
  launch_fold(st, kMaxBatch, fin, h->v64.xs, h->v64.xl, h->v64.x, h->P.n);
  double rr[kMaxBatch];
  true_residual(h, kMaxBatch, rr);
  launch_round(st, h->v64.xs, h->v64.xl, h->v64.tmp, h->P.n * kMaxBatch);
  unsigned restart = 0;
  std::vector<SReq *> finished;
  int64_t n = h->P.n, N = h->P.n_nodes;
  for (int k = 0; k < kMaxBatch; ++k) {
    if (!((fin >> k) & 1u)) continue;
    SSlot &sl = L.slot[k];
    SReq &q = *sl.req;
    double bb = hs.bnorm2[k];
    double rel;
    int status;
    if (bb == 0.0) {
      rel = 0.0;
      status = VEMG_OK;
    } else if (hs.status[k] == -6 || !std::isfinite(bb)) {
      rel = NAN;
      status = VEMG_ERR_BREAKDOWN;
    } else {
      rel = std::sqrt(rr[k] / bb);
      if (rel <= q.rtol) status = VEMG_OK;
      else if (hs.iters[k] >= q.max_iter) status = VEMG_WARN_MAXITER;
      else if (sl.restarts >= h->opt.max_restarts || rel > 0.5 * sl.prev) status = VEMG_WARN_FLOOR;
      else {
        sl.prev = rel;
        sl.restarts++;
        restart |= 1u << k;
        continue;
      }
    }
    double *xk = q.x + (int64_t)sl.col * N;
    launch_fill<double>(st, xk, N, 0.0, nullptr);
    launch_scatter(st, kMaxBatch, k, h->v64.tmp, h->perm, xk, n);
    q.iters[sl.col] = hs.iters[k];
    q.rel[sl.col] = rel;
    if (status < 0 || (q.status >= 0 && status > q.status)) q.status = status;
    if (--q.cols_left == 0) finished.push_back(&q);
    sl = SSlot();
    sv->cols_done++;
  }
  if (restart) lane_start(L, restart, true);
  HIPCHK(hipStreamSynchronize(st));
  for (SReq *q : finished) finish_request(sv, *q);
}

void server_loop(Server *sv) {
  (void)hipSetDevice(sv->device);
  while (true) {
    int precision;
    {
      std::unique_lock<std::mutex> lk(sv->mu);
      auto has_work = [&]() {
        if (!sv->incoming.empty()) return true;
        for (auto &L : sv->lanes)
          if (L->busy()) return true;
        return false;
      };
      sv->cv.wait(lk, [&]() { return sv->stop || has_work(); });
      if (sv->stop && !has_work()) break;
      while (!sv->incoming.empty()) {
        SReq *q = sv->incoming.front();
        sv->incoming.pop_front();
        for (int c = 0; c < q->nrhs; ++c) sv->lanes[q->mesh]->queue.emplace_back(q, c);
      }
      precision = sv->opt.precision;
    }
    try {
      // admission, joins and launches: every lane's chunk is queued before
      // any lane is waited on, so different meshes overlap on the device
      for (auto &Lp : sv->lanes) {
        Lane &L = *Lp;
        L.launched = false;
        if (!L.busy()) continue;
        if (!lane_admit(sv, L)) continue;
        L.last_used = ++sv->tick;
        // a precision switch waits for every request to finish, so a lane
        // that takes it is idle
        L.h->opt.precision = precision;
        unsigned mask = 0;
        for (int k = 0; k < kMaxBatch && !L.queue.empty(); ++k)
          if (!L.slot[k].req) {
            L.slot[k] = SSlot();
            L.slot[k].req = L.queue.front().first;
            L.slot[k].col = L.queue.front().second;
            L.queue.pop_front();
            mask |= 1u << k;
          }
        if (mask) lane_start(L, mask, false);
        int active = 0;
        for (auto &sl : L.slot) active += sl.req != nullptr;
        if (!active) continue;
        int kind = L.h->opt.precision != VEMG_FP64 ? kGraphMixedPC : kGraphFP64;
        run_chunk<double>(L.h, kMaxBatch, kind);
        HIPCHK(hipMemcpyAsync(L.scal_host, L.h->scal, sizeof(Scal), hipMemcpyDeviceToHost, L.h->work));
        HIPCHK(hipEventRecord(L.scal_ready, L.h->work));
        L.launched = true;
        sv->chunks++;
        sv->active_slots += active;
      }
      for (auto &Lp : sv->lanes)
        if (Lp->launched) lane_collect(sv, *Lp);
    } catch (const std::exception &e) {
      std::lock_guard<std::mutex> lk(sv->mu);
      sv->err = e.what();
      sv->stop = true;
      // fail every pending request so that waiters return
      for (auto &q : sv->reqs)
        if (!q->done) {
          q->done = true;
          q->status = VEMG_ERR_DEVICE;
          q->t_done = now_s();
          sv->completed.push_back(q.get());
        }
      for (auto &L : sv->lanes) {
        L->queue.clear();
        for (auto &sl : L->slot) sl = SSlot();
      }
      sv->incoming.clear();
      sv->cv_done.notify_all();
      break;
    }
  }
}

}  // namespace
}  // namespace vemg

namespace vemg {
namespace {

bool valid_options(const vemg_options &opt) {
  return !(opt.top_bc < 0 || opt.top_bc > 2 ||
           (opt.top_bc == VEMG_TOP_ROBIN && !(opt.robin_alpha > 0.0 && std::isfinite(opt.robin_alpha))) ||
           opt.pc < 0 || opt.pc > 5 || opt.max_levels < 1 || opt.max_levels > 16 || opt.coarse_max < 1 ||
           opt.coarse_max > 8192 || !(opt.theta >= 0.0) || opt.poll_every < 1 || opt.precision < 0 ||
           opt.precision > 2 || !(opt.inner_rtol > 0.0 && opt.inner_rtol < 1.0) || opt.max_outer < 1 ||
           opt.extrapolation < 0 || opt.extrapolation > 1);
}

// A handle on `device`.  pool == nullptr: the handle creates its own work
// stream; otherwise it runs on pool, which stays the caller's.
vemg_status create_handle(const vemg_options *o, int device, hipStream_t user, hipStream_t pool,
                          vemg_solver *out) {
  if (!out) return VEMG_ERR_INVALID_ARG;
  *out = nullptr;
  vemg_options opt;
  if (o)
    opt = *o;
  else
    vemg_default_options(&opt);
  if (!valid_options(opt)) return VEMG_ERR_INVALID_ARG;
  auto *h = new (std::nothrow) vemg_solver_s();
  if (!h) return VEMG_ERR_OOM;
  h->opt = opt;
  h->device = device;
  h->user = user;
  int st = guarded(h, [&]() -> int {
    if (device >= 0) {
      if (pool) {
        h->own_stream = false;
        h->work = pool;
      } else {
        HIPCHK(create_queue_stream(device, &h->work));
      }
      HIPCHK(hipEventCreateWithFlags(&h->ev, hipEventDisableTiming));
      HIPCHK(hipHostMalloc((void **)&h->host, sizeof(HostBox), hipHostMallocDefault));
    }
    return VEMG_OK;
  });
  if (st != VEMG_OK) {
    (void)vemg_destroy(h);  // releases whatever was created before the failure
    return (vemg_status)st;
  }
  *out = h;
  return VEMG_OK;
}

}  // namespace
}  // namespace vemg

using vemg::guarded;

extern "C" {

void vemg_default_options(vemg_options *o) {
  if (!o) return;
  o->top_bc = VEMG_TOP_PINNED;
  o->pin_node = -1;
  o->pc = VEMG_PC_VL_ADDITIVE;
  o->theta = 0.01;
  o->prolong_omega = 2.0 / 3.0;
  o->max_levels = 10;
  o->coarse_max = 8192;
  o->poll_every = 8;
  o->max_restarts = 5;
  o->use_graphs = 1;
  o->precision = VEMG_FP64;
  o->inner_rtol = 1e-4;
  o->max_outer = 30;
  o->robin_alpha = 0.0;
  o->extrapolation = VEMG_EXTRAP_PROJECTION;
}

vemg_status vemg_create(const vemg_options *o, int device, void *hip_stream, vemg_solver *out) {
  return vemg::create_handle(o, device, (hipStream_t)hip_stream, nullptr, out);
}

vemg_status vemg_setup(vemg_solver s, int64_t n_nodes, const double *xyz, int64_t n_tets, const int64_t *tets,
                       const uint8_t *top_mask) {
  if (!s) return VEMG_ERR_INVALID_ARG;
  return (vemg_status)guarded(s, [&]() -> int {
    s->ready = false;
    vemg::destroy_graphs(s);
    s->ar.release();
    vemg::SetupOptions so;
    so.top_dirichlet = s->opt.top_bc == VEMG_TOP_DIRICHLET;
    so.robin = s->opt.top_bc == VEMG_TOP_ROBIN;
    so.robin_alpha = s->opt.robin_alpha;
    so.build_sa = s->opt.pc == VEMG_PC_SA;
    so.extrapolation = s->opt.extrapolation;
    so.pin_node = s->opt.pin_node;
    so.theta = s->opt.theta;
    so.prolong_omega = s->opt.prolong_omega;
    so.max_levels = s->opt.max_levels;
    so.coarse_max = s->opt.coarse_max;
    s->P = vemg::Problem();
    vemg::build_problem(s->P, so, n_nodes, xyz, n_tets, tets, top_mask);
    s->footprint = vemg::count_upload_bytes(s);
    if (s->device >= 0) {
      vemg::upload(s);
      if (s->ar.bytes != s->footprint)
        throw vemg::DeviceError(VEMG_ERR_DEVICE, "device allocations differ from the counted footprint");
    }
    s->ready = true;
    s->err.clear();
    return VEMG_OK;
  });
}

vemg_status vemg_rhs(vemg_solver s, const double *f_host, double *b_host) {
  if (!s || !f_host || !b_host) return VEMG_ERR_INVALID_ARG;
  if (!s->ready) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int {
    vemg::mass_rhs(s->P, f_host, b_host);
    return VEMG_OK;
  });
}

vemg_status vemg_matvec(vemg_solver s, const double *x_dev, double *y_dev) {
  if (!s || !x_dev || !y_dev) return VEMG_ERR_INVALID_ARG;
  if (!s->ready || s->device < 0) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int {
    vemg::matvec(s, x_dev, y_dev, s->v64.tmp, s->v64.res);
    return VEMG_OK;
  });
}

vemg_status vemg_matvec_noalloc(vemg_solver s, const double *x_dev, double *y_dev) {
  if (!s || !x_dev || !y_dev) return VEMG_ERR_INVALID_ARG;
  if (!s->ready || s->device < 0) return VEMG_ERR_STATE;
  if (s->P.n > vemg::kScratchRows) {
    s->err = "vemg_matvec_noalloc: " + std::to_string(s->P.n) + " unknowns exceed the static buffer's " +
             std::to_string(vemg::kScratchRows);
    return VEMG_ERR_INVALID_ARG;
  }
  return (vemg_status)guarded(s, [&]() -> int {
    double *buf = vemg::scratch_of(s->device);  // [0, n): x in storage order; [n, 2n): A x
    vemg::matvec(s, x_dev, y_dev, buf, buf + s->P.n);
    return VEMG_OK;
  });
}

vemg_status vemg_solve(vemg_solver s, int nrhs, const double *b_dev, double *x_dev, double rtol, int max_iter,
                       int *iters, double *relres) {
  if (!s || !b_dev || !x_dev || nrhs < 1 || !(rtol >= 0.0) || max_iter < 1) return VEMG_ERR_INVALID_ARG;
  if (!s->ready || s->device < 0) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int { return vemg::do_solve(s, nrhs, b_dev, x_dev, rtol, max_iter, iters, relres); });
}

vemg_status vemg_apply(vemg_solver s, int op, const double *in_dev, double *out_dev) {
  if (!s || !in_dev || !out_dev) return VEMG_ERR_INVALID_ARG;
  if (!s->ready || s->device < 0) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int { return vemg::do_apply(s, op, in_dev, out_dev); });
}

vemg_status vemg_time_op(vemg_solver s, int op, int nrhs, int reps, double *avg_ms, int *launches) {
  if (!s || !avg_ms || reps < 1) return VEMG_ERR_INVALID_ARG;
  if (!s->ready || s->device < 0) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int { return vemg::do_time(s, op, nrhs, reps, avg_ms, launches); });
}

vemg_status vemg_set_preconditioner(vemg_solver s, int pc) {
  if (!s || pc < 0 || pc > 5) return VEMG_ERR_INVALID_ARG;
  if (pc == VEMG_PC_SA && s->P.SA.empty()) {
    s->err = "the smoothed aggregation baseline hierarchy is built only when the handle is set up with it";
    return VEMG_ERR_STATE;
  }
  return (vemg_status)guarded(s, [&]() -> int {
    if (s->device >= 0 && s->work) HIPCHK(hipStreamSynchronize(s->work));
    vemg::destroy_graphs(s);
    s->opt.pc = pc;
    return VEMG_OK;
  });
}

vemg_status vemg_set_precision(vemg_solver s, int precision) {
  if (!s || precision < 0 || precision > 2) return VEMG_ERR_INVALID_ARG;
  s->opt.precision = precision;
  return VEMG_OK;
}

vemg_status vemg_get_info(vemg_solver s, vemg_info *info) {
  if (!s || !info) return VEMG_ERR_INVALID_ARG;
  if (!s->ready) return VEMG_ERR_STATE;
  std::memset(info, 0, sizeof(*info));
  const vemg::Problem &P = s->P;
  info->n_nodes = P.n_nodes;
  info->n = P.n;
  info->n_top = P.n_top;
  info->pin_node = P.pin;
  info->nnz_offdiag = P.Aoff.nnz();
  info->s_levels = (int)P.S.size();
  info->abar_levels = (int)P.Abar.size();
  for (size_t l = 0; l < P.S.size() && l < 16; ++l) {
    info->s_rows[l] = P.S[l].n();
    info->s_nnz[l] = P.S[l].A.nnz() - P.S[l].n();
    info->p_nnz_s[l] = P.S[l].P.nnz();
  }
  for (size_t l = 0; l < P.Abar.size() && l < 16; ++l) {
    info->abar_rows[l] = P.Abar[l].n();
    info->abar_nnz[l] = P.Abar[l].A.nnz() - P.Abar[l].n();
    info->p_nnz_abar[l] = P.Abar[l].P.nnz();
  }
  info->e_nnz = P.E.nnz();
  info->fine_colours_top = (int)P.top_colour_start.size() - 1;
  info->fine_colours_bar = (int)P.bar_colour_start.size() - 1;
  info->device_bytes = s->ar.bytes;
  return VEMG_OK;
}

vemg_status vemg_footprint(vemg_solver s, int nrhs, size_t *bytes) {
  if (!s || !bytes || nrhs < 0) return VEMG_ERR_INVALID_ARG;
  if (!s->ready) return VEMG_ERR_STATE;
  *bytes = s->footprint + (size_t)2 * (size_t)nrhs * (size_t)s->P.n_nodes * sizeof(double);
  return VEMG_OK;
}

vemg_status vemg_export(vemg_solver s, const char *name, void *buf, size_t *bytes) {
  if (!s || !name || !bytes) return VEMG_ERR_INVALID_ARG;
  if (!s->ready) return VEMG_ERR_STATE;
  return (vemg_status)guarded(s, [&]() -> int { return vemg::do_export(s, name, buf, bytes); });
}

vemg_status vemg_destroy(vemg_solver s) {
  if (!s) return VEMG_ERR_INVALID_ARG;
  if (s->device >= 0) {
    (void)hipSetDevice(s->device);
    if (s->work) (void)hipStreamSynchronize(s->work);
    vemg::destroy_graphs(s);
    s->ar.release();
    if (s->ev) (void)hipEventDestroy(s->ev);
    if (s->own_stream && s->work) (void)hipStreamDestroy(s->work);
    if (s->host) (void)hipHostFree(s->host);
  }
  delete s;
  return VEMG_OK;
}

const char *vemg_status_string(vemg_status st) {
  switch (st) {
    case VEMG_OK: return "ok";
    case VEMG_WARN_MAXITER: return "maximum iteration count reached";
    case VEMG_WARN_FLOOR: return "true residual stalled above the tolerance";
    case VEMG_ERR_INVALID_ARG: return "invalid argument";
    case VEMG_ERR_MESH: return "invalid mesh";
    case VEMG_ERR_PROJECTION: return "node does not project onto the top surface";
    case VEMG_ERR_OOM: return "out of memory";
    case VEMG_ERR_DEVICE: return "device error";
    case VEMG_ERR_BREAKDOWN: return "CG breakdown (p.Ap <= 0 or not finite)";
    case VEMG_ERR_STATE: return "call out of order";
  }
  return "unknown status";
}

const char *vemg_last_error(vemg_solver s) { return s ? s->err.c_str() : ""; }


vemg_status vemg_server_create(int device, size_t hbm_budget, const vemg_options *o, vemg_server *out) {
  if (!out || device < 0) return VEMG_ERR_INVALID_ARG;
  *out = nullptr;
  vemg_options opt;
  if (o)
    opt = *o;
  else
    vemg_default_options(&opt);
  if (!vemg::valid_options(opt)) return VEMG_ERR_INVALID_ARG;
  auto *sv = new (std::nothrow) vemg_server_s();
  if (!sv) return VEMG_ERR_OOM;
  sv->opt = opt;
  if (sv->opt.precision == VEMG_MIXED_IR) sv->opt.precision = VEMG_MIXED_PC;
  sv->device = device;
  sv->budget = hbm_budget;
  hipError_t e = hipSetDevice(device);
  for (int i = 0; e == hipSuccess && i < vemg::kServerStreams; ++i)
    e = vemg::create_queue_stream(device, &sv->streams[i]);
  if (e != hipSuccess) {
    (void)vemg_server_destroy(sv);
    return e == hipErrorOutOfMemory ? VEMG_ERR_OOM : VEMG_ERR_DEVICE;
  }
  *out = sv;
  return VEMG_OK;
}

vemg_status vemg_server_add_mesh(vemg_server sv, int64_t n_nodes, const double *xyz, int64_t n_tets,
                                 const int64_t *tets, const uint8_t *top_mask, int *mesh_id) {
  if (!sv || !mesh_id) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  if (sv->started) {
    sv->err = "meshes must be added before the first submit";
    return VEMG_ERR_STATE;
  }
  const int lane = (int)sv->lanes.size();
  vemg_solver h = nullptr;
  vemg_status st = vemg::create_handle(&sv->opt, sv->device, nullptr, sv->streams[lane % vemg::kServerStreams], &h);
  if (st != VEMG_OK) return st;
  // a mesh that alone exceeds the budget is refused before its upload
  auto L = std::make_unique<vemg::Lane>();
  L->h = h;
  int gst = guarded(h, [&]() -> int {
    h->device = -1;  // host setup only: the footprint is counted, nothing uploaded yet
    vemg_status s2 = vemg_setup(h, n_nodes, xyz, n_tets, tets, top_mask);
    h->device = sv->device;
    if (s2 != VEMG_OK) return s2;
    HIPCHK(hipSetDevice(sv->device));
    L->footprint = h->footprint;
    if (sv->budget && L->footprint > sv->budget) {
      h->err = "mesh needs more device memory than the budget";
      return VEMG_ERR_OOM;
    }
    HIPCHK(hipHostMalloc((void **)&L->scal_host, sizeof(vemg::Scal), hipHostMallocDefault));
    HIPCHK(hipEventCreateWithFlags(&L->scal_ready, hipEventDisableTiming));
    if (sv->budget && sv->used + L->footprint > sv->budget) return VEMG_OK;  // uploaded when needed
    vemg::upload(h);
    if (h->ar.bytes != L->footprint)
      throw vemg::DeviceError(VEMG_ERR_DEVICE, "device allocations differ from the counted footprint");
    // capture both precisions' graphs now, while no other thread uses the device
    if (h->opt.use_graphs) {
      const int unit = vemg::chunk_unit(h->opt.poll_every);
      vemg::iteration_graph<double>(h, vemg::kMaxBatch, vemg::kGraphFP64, unit, true);
      vemg::iteration_graph<double>(h, vemg::kMaxBatch, vemg::kGraphMixedPC, unit, true);
      HIPCHK(hipStreamSynchronize(h->work));
    }
    L->resident = true;
    sv->used += L->footprint;
    sv->uploads++;
    return VEMG_OK;
  });
  h->allow_capture = false;
  if (gst != VEMG_OK) {
    sv->err = h->err;
    if (L->scal_host) (void)hipHostFree(L->scal_host);
    if (L->scal_ready) (void)hipEventDestroy(L->scal_ready);
    vemg_destroy(h);
    return (vemg_status)gst;
  }
  *mesh_id = lane;
  sv->lanes.push_back(std::move(L));
  return VEMG_OK;
}

vemg_status vemg_server_rhs(vemg_server sv, int mesh_id, const double *f_host, double *b_host) {
  if (!sv) return VEMG_ERR_INVALID_ARG;
  vemg_solver h;
  {
    std::lock_guard<std::mutex> lk(sv->mu);
    if (mesh_id < 0 || mesh_id >= (int)sv->lanes.size()) return VEMG_ERR_INVALID_ARG;
    h = sv->lanes[mesh_id]->h;
  }
  return vemg_rhs(h, f_host, b_host);  // host arithmetic on the immutable host setup
}

vemg_status vemg_server_footprint(vemg_server sv, int mesh_id, int nrhs, size_t *bytes) {
  if (!sv) return VEMG_ERR_INVALID_ARG;
  vemg_solver h;
  {
    std::lock_guard<std::mutex> lk(sv->mu);
    if (mesh_id < 0 || mesh_id >= (int)sv->lanes.size()) return VEMG_ERR_INVALID_ARG;
    h = sv->lanes[mesh_id]->h;
  }
  return vemg_footprint(h, nrhs, bytes);  // reads the footprint fixed at setup
}

vemg_status vemg_server_submit(vemg_server sv, int mesh_id, int nrhs, const double *b_dev, double *x_dev, double rtol,
                               int max_iter, uint64_t *req_id) {
  if (!sv || !b_dev || !x_dev || nrhs < 1 || !(rtol >= 0.0) || max_iter < 1) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  if (mesh_id < 0 || mesh_id >= (int)sv->lanes.size()) return VEMG_ERR_INVALID_ARG;
  if (sv->stop) return VEMG_ERR_STATE;
  if (!sv->started) {
    sv->started = true;
    sv->worker = std::thread(vemg::server_loop, sv);
  }
  auto q = std::make_unique<vemg::SReq>();
  q->id = sv->next_id++;
  q->mesh = mesh_id;
  q->nrhs = nrhs;
  q->b = b_dev;
  q->x = x_dev;
  q->rtol = rtol;
  q->max_iter = std::min(max_iter, 1 << 20);
  q->t_submit = vemg::now_s();
  q->cols_left = nrhs;
  q->iters.assign(nrhs, 0);
  q->rel.assign(nrhs, 0.0);
  if (sv->first_submit < 0) sv->first_submit = q->t_submit;
  if (req_id) *req_id = q->id;
  sv->by_id[q->id] = q.get();
  sv->incoming.push_back(q.get());
  sv->reqs.push_back(std::move(q));
  sv->cv.notify_all();
  return VEMG_OK;
}

vemg_status vemg_server_poll(vemg_server sv, uint64_t *done_ids, int cap, int *n_done) {
  if (!sv || !n_done || (cap > 0 && !done_ids)) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  int k = 0;
  while (k < cap && !sv->completed.empty()) {
    done_ids[k++] = sv->completed.front()->id;
    sv->completed.pop_front();
  }
  *n_done = k;
  return sv->err.empty() ? VEMG_OK : VEMG_ERR_DEVICE;
}

vemg_status vemg_server_wait(vemg_server sv, uint64_t req_id, double timeout_s) {
  if (!sv) return VEMG_ERR_INVALID_ARG;
  std::unique_lock<std::mutex> lk(sv->mu);
  auto it = sv->by_id.find(req_id);
  if (it == sv->by_id.end()) return VEMG_ERR_INVALID_ARG;
  vemg::SReq *q = it->second;
  auto pred = [&]() { return q->done; };
  if (timeout_s > 0) {
    if (!sv->cv_done.wait_for(lk, std::chrono::duration<double>(timeout_s), pred)) return VEMG_ERR_STATE;
  } else {
    sv->cv_done.wait(lk, pred);
  }
  return sv->err.empty() ? VEMG_OK : VEMG_ERR_DEVICE;
}

vemg_status vemg_server_result(vemg_server sv, uint64_t req_id, int *status, int *iters, double *relres,
                               double *latency_ms) {
  if (!sv) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  auto it = sv->by_id.find(req_id);
  if (it == sv->by_id.end()) return VEMG_ERR_INVALID_ARG;
  const vemg::SReq &q = *it->second;
  if (!q.done) return VEMG_ERR_STATE;
  if (status) *status = q.status;
  for (int c = 0; c < q.nrhs; ++c) {
    if (iters) iters[c] = q.iters[c];
    if (relres) relres[c] = q.rel[c];
  }
  if (latency_ms) *latency_ms = 1e3 * (q.t_done - q.t_submit);
  return VEMG_OK;
}

vemg_status vemg_server_get_stats(vemg_server sv, vemg_server_stats *st) {
  if (!sv || !st) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  std::memset(st, 0, sizeof(*st));
  std::vector<double> lat;
  int64_t pending = 0;
  for (size_t i = (size_t)sv->reqs_base; i < sv->reqs.size(); ++i) {
    if (sv->reqs[i]->done) lat.push_back(1e3 * (sv->reqs[i]->t_done - sv->reqs[i]->t_submit));
    else ++pending;
  }
  std::sort(lat.begin(), lat.end());
  st->requests_done = (int64_t)lat.size();
  st->requests_queued = pending;
  st->columns_done = sv->cols_done;
  if (!lat.empty()) {
    auto pct = [&](double p) {
      double pos = p * (double)(lat.size() - 1);
      size_t i = (size_t)pos;
      double f = pos - (double)i;
      return i + 1 < lat.size() ? lat[i] * (1.0 - f) + lat[i + 1] * f : lat[i];
    };
    st->p50_ms = pct(0.50);
    st->p99_ms = pct(0.99);
    double sum = 0.0;
    for (double v : lat) sum += v;
    st->mean_ms = sum / (double)lat.size();
    st->max_ms = lat.back();
  }
  if (sv->last_done > sv->first_submit && sv->first_submit >= 0) {
    st->busy_s = sv->last_done - sv->first_submit;
    st->solves_per_s = (double)st->columns_done / st->busy_s;
  }
  const int64_t chunks = sv->chunks;
  st->mean_slot_occupancy = chunks ? (double)sv->active_slots / (double)(chunks * vemg::kMaxBatch) : 0.0;
  st->chunks = chunks;
  st->uploads = sv->uploads;
  st->evictions = sv->evictions;
  st->resident_bytes = sv->used;
  st->budget_bytes = sv->budget;
  return VEMG_OK;
}

vemg_status vemg_server_set_precision(vemg_server sv, int precision) {
  if (!sv || precision < 0 || precision > 2) return VEMG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(sv->mu);
  if (!sv->incoming.empty()) return VEMG_ERR_STATE;
  for (auto &q : sv->reqs)
    if (!q->done) return VEMG_ERR_STATE;
  // every request is done: the scheduler holds no slot and applies the new
  // precision to a lane before its next chunk
  sv->opt.precision = precision == VEMG_MIXED_IR ? VEMG_MIXED_PC : precision;
  sv->first_submit = sv->last_done = -1.0;
  sv->chunks = 0;
  sv->cols_done = 0;
  sv->active_slots = 0;
  for (auto &q : sv->reqs) q->t_done = q->t_submit = 0.0;
  sv->reqs_base = (int64_t)sv->reqs.size();
  return VEMG_OK;
}

vemg_status vemg_server_destroy(vemg_server sv) {
  if (!sv) return VEMG_ERR_INVALID_ARG;
  {
    std::lock_guard<std::mutex> lk(sv->mu);
    sv->stop = true;
    sv->cv.notify_all();
  }
  if (sv->worker.joinable()) sv->worker.join();
  (void)hipSetDevice(sv->device);
  for (auto &L : sv->lanes) {
    vemg_destroy(L->h);
    if (L->scal_host) (void)hipHostFree(L->scal_host);
    if (L->scal_ready) (void)hipEventDestroy(L->scal_ready);
  }
  for (hipStream_t st : sv->streams)
    if (st) (void)hipStreamDestroy(st);
  delete sv;
  return VEMG_OK;
}

const char *vemg_server_last_error(vemg_server sv) { return sv ? sv->err.c_str() : ""; }

}  // extern "C"
