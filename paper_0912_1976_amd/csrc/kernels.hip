// HIP kernels of the PCG hot path for gfx950 (CDNA4, wave64).
//
// The path is sparse: every kernel streams its matrix once with coalesced loads
// (SELL-64 for the fine operator, CSR rows over groups of lanes for coarse
// operators and transfers), reads each matrix entry once for all K right-hand
// sides of a batch, gathers the vector rows it needs through L2 / the Infinity
// Cache, and keeps reductions deterministic (per-block partials, added in an
// order that does not depend on K).  The matrix cores multiply by the dense
// triangular factors of the coarse levels' patches.  Blocks are renumbered so
// that each of the eight XCDs works on a contiguous range of rows, which keeps
// the gathered vector lines in that XCD's L2.
#include <type_traits>

#include "kernels.hpp"

namespace vemg {

namespace {

// Hardware dispatches block b to XCD b % 8; give every XCD a contiguous chunk.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
  int64_t q = nb >> 3, rem = nb & 7, x = b & 7, i = b >> 3;
  return (x < rem) ? x * (q + 1) + i : rem * (q + 1) + (x - rem) * q + i;
}

// Every kernel of an iteration leaves at once when all columns are done.  The
// flag is read beside the kernel's first loads, which `keep` holds in front of
// the branch on it: read on its own it puts a trip to memory ahead of them.
__device__ const int kNeverDone = 0;
__device__ __forceinline__ int stop_flag(const int *done) { return *(done ? done : &kNeverDone); }
__device__ __forceinline__ void keep() {}
template <class V, class... W>
__device__ __forceinline__ void keep(const V &v, const W &...w) {
  asm volatile("" ::"v"(v));
  keep(w...);
}

template <class T, int K>
struct alignas(sizeof(T) * K) Row {
  T v[K];
};

template <class T, int K>
__device__ __forceinline__ Row<T, K> ld(const T *__restrict__ p, int64_t r) {
  return *reinterpret_cast<const Row<T, K> *>(p + r * K);
}
template <class T, int K>
__device__ __forceinline__ void st(T *__restrict__ p, int64_t r, const Row<T, K> &v) {
  *reinterpret_cast<Row<T, K> *>(p + r * K) = v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sums v[0..K) over a 256-thread block in a fixed order and writes the K
// results to out[0..K) (thread 0).  Every thread of the block must call it.
template <int K>
__device__ __forceinline__ void block_sum_store(const double (&v)[K], double *out) {
  __shared__ double red[kSlicesPerBlock][kMaxBatch];
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double t = wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) red[w][k] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < kSlicesPerBlock; ++q) t += red[q][k];
      out[k] = t;
    }
  }
}

// v + the value of lane (own lane xor D), D a power of two, in a few vector
// instructions (a shuffle through LDS costs a pass of the LDS per word: at
// K = 8 the reductions by shuffles took most of the restriction's time)
template <int D>
__device__ __forceinline__ int lane_xor(int v) {
  static_assert(D == 1 || D == 2 || D == 4 || D == 8, "lane_xor");
  if constexpr (D == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
  if constexpr (D == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
  if constexpr (D == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);  // row_ror 8
  if constexpr (D == 4) {
    const int t = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);  // row_shl 4 in the even banks
    return __builtin_amdgcn_update_dpp(t, v, 0x114, 0xf, 0xa, false);         // row_shr 4 in the odd ones
  }
}
// cache policy of loads and stores at agent scope on gfx950 (sc1)
constexpr int kAgentScope = 16;

template <class T, int N>
struct Words {
  int w[N];
};
template <int D, class T>
__device__ __forceinline__ T add_xor(T v) {
  constexpr int N = sizeof(T) / 4;
  const auto a = __builtin_bit_cast(Words<T, N>, v);
  Words<T, N> p, q = a;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (D == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap((unsigned)a.w[i], (unsigned)a.w[i], false, false);
      q.w[i] = r[0];
      p.w[i] = r[1];
    } else if constexpr (D == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap((unsigned)a.w[i], (unsigned)a.w[i], false, false);
      q.w[i] = r[0];
      p.w[i] = r[1];
    } else {
      p.w[i] = lane_xor<D>(a.w[i]);
    }
  }
  return __builtin_bit_cast(T, q) + __builtin_bit_cast(T, p);
}

// Sums v over the 64 rows of a block of 64 LPR threads (LPR lanes a row) into
// out[0..K): adjacent rows first, then pairs of pairs and so on, the same tree
// for every LPR.  Every thread of the block must call it.
template <int D>
__device__ __forceinline__ double rows_tree(double v) {
  if constexpr (D < kWave)
    return rows_tree<2 * D>(add_xor<D>(v));
  else
    return v;
}
template <int K, int LPR>
__device__ __forceinline__ void slice_sum_store(const double (&v)[K / LPR], double *out) {
  constexpr int C = K / LPR;
  double t[C];
#pragma unroll
  for (int k = 0; k < C; ++k) t[k] = rows_tree<LPR>(v[k]);
  const int lane = threadIdx.x & 63;
  if constexpr (LPR == 1) {
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < C; ++k) out[k] = t[k];
    }
  } else {
    __shared__ double red[LPR][K];
    if (lane < LPR) {
#pragma unroll
      for (int k = 0; k < C; ++k) red[threadIdx.x >> 6][lane * C + k] = t[k];
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < K) {
      if constexpr (LPR == 4)
        out[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
      else
        out[k] = red[0][k] + red[1][k];
    }
  }
}

template <class T>
__device__ __forceinline__ const T *sell_vals(const Sell &A);
template <>
__device__ __forceinline__ const double *sell_vals<double>(const Sell &A) {
  return A.val64;
}
template <>
__device__ __forceinline__ const float *sell_vals<float>(const Sell &A) {
  return A.val32;
}
template <class T>
__device__ __forceinline__ const T *csr_vals(const CsrG &A);
template <>
__device__ __forceinline__ const double *csr_vals<double>(const CsrG &A) {
  return A.val64;
}
template <>
__device__ __forceinline__ const float *csr_vals<float>(const CsrG &A) {
  return A.val32;
}

// Lanes that share one row of a K-column batch in the fine kernels: each
// lane holds CPL = K / LPR consecutive columns, 16 bytes at most, so that a
// gathered row is one 16-byte load per lane and the LPR lanes of a row read
// it contiguously.  Narrow rows keep one lane per row.  Spreading a wide row
// over lanes keeps the registers per lane small and several gathers in
// flight per lane, where a 64-byte row per lane allowed one.
template <class T, int K>
constexpr int row_lanes() {
  return sizeof(T) * K <= 16 ? 1 : (int)(sizeof(T) * K / 16);
}

// entries of a row kept in flight per lane
template <class T, int C>
constexpr int sell_unroll() {
  return sizeof(T) * C >= 64 ? 1 : sizeof(T) * C >= 32 ? 2 : 4;
}

// value of lane O of every group of LPR consecutive lanes (2 or 4) in all of them
template <int LPR, int O>
__device__ __forceinline__ int group_bcast(int v) {
  constexpr int ctrl = LPR == 4 ? O * 0x55 : O | O << 2 | (2 + O) << 4 | (2 + O) << 6;  // quad_perm
  return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, true);
}
template <int LPR, int O>
__device__ __forceinline__ float group_bcast(float v) {
  return __builtin_bit_cast(float, group_bcast<LPR, O>(__builtin_bit_cast(int, v)));
}
template <int LPR, int O>
__device__ __forceinline__ double group_bcast(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(group_bcast<LPR, O>(w.x), group_bcast<LPR, O>(w.y)));
}

// entry u of a step is lane u % LPR's u / LPR-th
template <int LPR, class T, int N>
__device__ __forceinline__ void spread(const int32_t (&c)[N], const T (&v)[N], int32_t (&cu)[N * LPR],
                                       T (&vu)[N * LPR]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    cu[i * LPR] = group_bcast<LPR, 0>(c[i]);
    vu[i * LPR] = group_bcast<LPR, 0>(v[i]);
    cu[i * LPR + 1] = group_bcast<LPR, 1>(c[i]);
    vu[i * LPR + 1] = group_bcast<LPR, 1>(v[i]);
    if constexpr (LPR == 4) {
      cu[i * LPR + 2] = group_bcast<LPR, 2>(c[i]);
      vu[i * LPR + 2] = group_bcast<LPR, 2>(v[i]);
      cu[i * LPR + 3] = group_bcast<LPR, 3>(c[i]);
      vu[i * LPR + 3] = group_bcast<LPR, 3>(v[i]);
    }
  }
}

// Off-diagonal terms of one SELL row, entries [begin, end) of its slice at
// position t, for the C columns [q C, q C + C) of a K-column batch:
// acc = sum_j v_j (x_j - x_r) (DIFF) or sum_j v_j x_j.  Every column is summed
// in storage order, whatever C is.  With OWN the entries pointing at row `own`
// itself (the padding of the L part, whose value the sweep has not written
// yet) count a zero.
// With several lanes a row, each lane loads every LPR-th entry's column and
// value for the others too, and those of the next four entries before the
// current ones' gathers; loaded by every lane they were two of the three
// loads an entry.  At K = 8 and 2,179,616 unknowns the prolongation between the
// sweeps went from 221 to 143 us, the forward sweep from 218 to 195, the
// residual from 174 to 153 and the product from 268 to 254.
template <class T, int K, int C, bool DIFF, bool OWN = false>
__device__ __forceinline__ void sell_span(const Sell &A, int64_t begin, int64_t end, int t, int q,
                                          const T *__restrict__ x, const Row<T, C> &xr, T (&acc)[C],
                                          int32_t own = -1) {
  constexpr int LPR = K / C;
  const int len = (int)((end - begin) >> 6);
  const int32_t *__restrict__ cp = A.col + begin + t;
  const T *__restrict__ vp = sell_vals<T>(A) + begin + t;
  const T *__restrict__ xq = x + q * C;
#pragma unroll
  for (int k = 0; k < C; ++k) acc[k] = T(0);
  auto row = [&](int32_t c) {
    Row<T, C> xc = *reinterpret_cast<const Row<T, C> *>(xq + (int64_t)c * K);
    if constexpr (OWN) {
#pragma unroll
      for (int k = 0; k < C; ++k) xc.v[k] = c != own ? xc.v[k] : T(0);
    }
    return xc;
  };
  auto add = [&](T v, const Row<T, C> &xc) {
#pragma unroll
    for (int k = 0; k < C; ++k) acc[k] += DIFF ? v * (xc.v[k] - xr.v[k]) : v * xc.v[k];
  };
  if constexpr (LPR == 1) {
    constexpr int U = sell_unroll<T, C>();
#pragma unroll U
    for (int e = 0; e < len; ++e) add(vp[(int64_t)e * 64], row(cp[(int64_t)e * 64]));
  } else {
    constexpr int U = 4, N = U / LPR;  // entries a step, and of those this lane's
    int32_t c[N];
    T v[N];
    auto load = [&](int e0) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int e = e0 + i * LPR + q;
        c[i] = e < len ? cp[(int64_t)e * 64] : 0;
        v[i] = e < len ? vp[(int64_t)e * 64] : T(0);
      }
    };
    load(0);
    for (int e0 = 0; e0 < len; e0 += U) {
      int32_t cu[U];
      T vu[U];
      spread<LPR>(c, v, cu, vu);
      load(e0 + U);
      Row<T, C> xc[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e0 + u < len) xc[u] = row(cu[u]);  // uniform over the slice
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e0 + u < len) add(vu[u], xc[u]);
    }
  }
}

// columns [q C, q C + C) of row r
template <class T, int K, int C>
__device__ __forceinline__ Row<T, C> ldp(const T *__restrict__ p, int64_t r, int q) {
  return *reinterpret_cast<const Row<T, C> *>(p + r * K + q * C);
}
template <class T, int K, int C>
__device__ __forceinline__ void stp(T *__restrict__ p, int64_t r, int q, const Row<T, C> &v) {
  *reinterpret_cast<Row<T, C> *>(p + r * K + q * C) = v;
}

// Block sums of per-row products when a row's K columns are spread over LPR
// lanes (blocks of kBlock * LPR threads covering kBlock rows): the products
// are first laid out one row per thread of the block's first kBlock threads,
// which then reduce exactly as block_sum_store does, so every column's sum
// has the same rounding as with one lane per row.  Every thread of the block
// must call it.
template <int K, int LPR>
__device__ __forceinline__ void block_sum_rows(const double (&v)[K / LPR], double *out) {
  constexpr int C = K / LPR;
  if constexpr (LPR == 1) {
    block_sum_store<K>(v, out);
  } else {
    __shared__ double buf[kBlock][K];
    const int rloc = threadIdx.x / LPR, q = threadIdx.x % LPR;
#pragma unroll
    for (int j = 0; j < C; ++j) buf[rloc][q * C + j] = v[j];
    __syncthreads();
    __shared__ double red[kSlicesPerBlock][kMaxBatch];
    if (threadIdx.x < kBlock) {  // whole wavefronts: wavefront w holds the rows of slice w
      const int w = threadIdx.x >> 6;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double t = wave_sum(buf[threadIdx.x][k]);
        if ((threadIdx.x & 63) == 0) red[w][k] = t;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kSlicesPerBlock; ++w) t += red[w][k];
        out[k] = t;
      }
    }
  }
}

// ------------------------------------------------------------- fine matrix
// (A x)_r in difference form, columns [q C, q C + C); the row's own operands
// are loaded before its entries
template <class T, int K, int C>
__device__ __forceinline__ Row<T, C> fine_row(const Sell &A, const SliceRef &S, int t, int q, int64_t r,
                                              const T *__restrict__ x, const Row<T, C> &xr) {
  T d0, d1 = T(0);
  if constexpr (std::is_same<T, double>::value) {
    d0 = A.d64[r];
  } else {
    d0 = A.s32[r];
    d1 = A.dh32[r];
  }
  T acc[C];
  sell_span<T, K, C, true>(A, S.begin, S.end, t, q, x, xr, acc);
  Row<T, C> out;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    if constexpr (std::is_same<T, double>::value)
      out.v[k] = acc[k] + d0 * xr.v[k];
    else
      out.v[k] = d0 * (acc[k] + d1 * xr.v[k]);
  }
  return out;
}

// y_r = -(V x)_r by lane q of row r's lanes, V the entries [begin, end) of row
// mi's slice (U: the residual after the forward sweep).
// Bandwidth and gathers bound it, and U holds half of the row: with the
// forward sweep reading L alone and this product U alone, FP64 solves of
// 2,179,616 unknowns went from 314.2 to 293.1 ms (eight right-hand sides) and
// from 123.8 to 115.6 ms (one).  On the same inputs one application of the
// preconditioner moved by 2e-16 (relative), at aspect ratios 1e-2 to 1e-4.
template <class T, int K>
__device__ __forceinline__ void residual_row(const Sell &A, int64_t begin, int64_t end, int64_t mi, int64_t r, int q,
                                             const T *__restrict__ x, T *y) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  T s0 = T(1);
  if constexpr (!std::is_same<T, double>::value) s0 = A.s32[mi];
  Row<T, C> out{};
  T acc[C];
  sell_span<T, K, C, false>(A, begin, end, (int)(mi & 63), q, x, out, acc);
#pragma unroll
  for (int k = 0; k < C; ++k) out.v[k] = -s0 * acc[k];
  stp<T, K, C>(y, r, q, out);
}

// Blocks of kBlock rows (four slices), row_lanes<T, K>() lanes per row.
// order: the range's slices in visit order; the blocks of one XCD take a
// contiguous part of it.
template <class T, int K, int MODE, bool DOT>
__global__ __launch_bounds__((kBlock * row_lanes<T, K>())) void k_spmv(
    Sell A, int64_t r0, int64_t r1, int64_t ns, int64_t nb, const SliceRef *__restrict__ order,
    const T *__restrict__ x, T *__restrict__ y, double *__restrict__ partial, const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  static_assert(!(MODE == 1 && DOT), "the residual form has no block reduction");
  const int stop = stop_flag(done);
  const int64_t blk = xcd_block(blockIdx.x, nb);
  const int rloc = threadIdx.x / LPR, q = threadIdx.x % LPR;
  const int t = rloc & 63;
  const int64_t i = blk * kSlicesPerBlock + __builtin_amdgcn_readfirstlane(rloc >> 6);
  SliceRef S{0, 0, 0, 0};
  if (i < ns) S = order[i];
  keep(S.end);
  if (stop) return;
  const int64_t r = S.slice * 64 + t;
  double prod[C];
#pragma unroll
  for (int k = 0; k < C; ++k) prod[k] = 0.0;
  if (i < ns && r >= r0 && r < r1) {
    if constexpr (MODE == 1) {
      // no block reduction in this form, so the lane may leave
      residual_row<T, K>(A, S.mid, S.end, r, r, q, x, y);
      return;
    }
    const Row<T, C> xr = ldp<T, K, C>(x, r, q);
    const Row<T, C> out = fine_row<T, K, C>(A, S, t, q, r, x, xr);
    stp<T, K, C>(y, r, q, out);
    if (DOT) {
#pragma unroll
      for (int k = 0; k < C; ++k) prod[k] = (double)xr.v[k] * (double)out.v[k];
    }
  }
  if (DOT) block_sum_rows<K, LPR>(prod, partial + blk * K);
}

// device form of the row ranges of one multicolour step
template <class T>
struct GsDev {
  int64_t r0[2], r1[2], sf[2], nb[2];
  T *x;
  int n;
  int64_t nbt;
};

// One Gauss-Seidel step of row r by lane q of its row_lanes<T, K>() lanes
// (columns [q C, q C + C)) with the right-hand side gs g_gi: x_r +
// (gs g - (A x)_r) / a_rr, or with FIRST (g - (L x)_r) / a_rr, the first
// sweep's step from zero, which reads L alone.  [begin, end): the entries of the row's slice (its L entries).
// prod: g x of the row.
// (mi: the row's index in A; r and gi: its index in x and in g)
template <class T, int K, bool FIRST>
__device__ __forceinline__ void gs_row(const Sell &A, int64_t begin, int64_t end, int64_t mi, int64_t r, int64_t gi,
                                       T gs, int q, const T *__restrict__ g, T *x,
                                       double (&prod)[K / row_lanes<T, K>()]) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  const int t = (int)(mi & 63);
  Row<T, C> xr{};
  if constexpr (!FIRST) xr = ldp<T, K, C>(x, r, q);
  const Row<T, C> gr = ldp<T, K, C>(g, gi, q);
  T d = T(0), i0;
  if constexpr (std::is_same<T, double>::value) {
    i0 = A.i64[mi];
    if (!FIRST) d = A.d64[mi];
  } else {
    i0 = 1.0f / A.s32[mi];  // the row-scaled operator has a unit diagonal
    if (!FIRST) d = A.dh32[mi];
  }
  T acc[C];
  sell_span<T, K, C, !FIRST, FIRST>(A, begin, end, t, q, x, xr, acc, (int32_t)r);
  Row<T, C> out;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    if constexpr (std::is_same<T, double>::value)
      out.v[k] = xr.v[k] + (gs * gr.v[k] - (acc[k] + d * xr.v[k])) * i0;
    else
      out.v[k] = xr.v[k] + (gs * gr.v[k] * i0 - (acc[k] + d * xr.v[k]));
    prod[k] = (double)gr.v[k] * (double)out.v[k];
  }
  stp<T, K, C>(x, r, q, out);
}

// The backward step of top row r of the merged cycles: as gs_row, its non-top
// neighbours' values taken as w - u (MergedRows).
template <class T, int K>
__device__ __forceinline__ void gs_top_row(const Sell &A, int64_t r, int q, const T *__restrict__ g, T *x,
                                           double (&prod)[K / row_lanes<T, K>()]) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  const int64_t s = r >> 6, base = A.sptr[s];
  const int t = (int)(r & 63), len = (int)((A.sptr[s + 1] - base) >> 6);
  const Row<T, C> xr = ldp<T, K, C>(x, r, q), gr = ldp<T, K, C>(g, r, q);
  T d, i0;
  if constexpr (std::is_same<T, double>::value) {
    i0 = A.i64[r];
    d = A.d64[r];
  } else {
    i0 = 1.0f / A.s32[r];
    d = A.dh32[r];
  }
  T acc[C];
#pragma unroll
  for (int k = 0; k < C; ++k) acc[k] = T(0);
#pragma unroll 2
  for (int e = 0; e < len; ++e) {
    const int64_t p = base + t + (int64_t)e * 64;
    const int32_t c = A.col[p], cu = A.col2[p];
    const T v = sell_vals<T>(A)[p];
    const Row<T, C> xc = ldp<T, K, C>(x, c, q), uc = ldp<T, K, C>(x, cu < 0 ? c : cu, q);
#pragma unroll
    for (int k = 0; k < C; ++k) acc[k] += v * ((xc.v[k] - (cu < 0 ? T(0) : uc.v[k])) - xr.v[k]);
  }
  Row<T, C> out;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    if constexpr (std::is_same<T, double>::value)
      out.v[k] = xr.v[k] + (gr.v[k] - (acc[k] + d * xr.v[k])) * i0;
    else
      out.v[k] = xr.v[k] + (gr.v[k] * i0 - (acc[k] + d * xr.v[k]));
    prod[k] = (double)gr.v[k] * (double)out.v[k];
  }
  stp<T, K, C>(x, r, q, out);
}

// the slice of block b (of J.nbt) and its rows of the range
struct GsSlice {
  int64_t s, r0, r1;
};
template <class T>
__device__ __forceinline__ GsSlice gs_slice(const GsDev<T> &J, int64_t b) {
  int64_t blk = xcd_block(b, J.nbt);
  const bool second = J.n > 1 && blk >= J.nb[0];
  if (second) blk -= J.nb[0];
  return second ? GsSlice{J.sf[1] + blk, J.r0[1], J.r1[1]} : GsSlice{J.sf[0] + blk, J.r0[0], J.r1[0]};
}

// one slice per block (a colour holds few rows, so small blocks spread them
// over every CU), row_lanes<T, K>() lanes per row; up to two row ranges (the
// top and the non-top rows of one colour)
template <class T, int K, bool FIRST>
__global__ __launch_bounds__((kWave * row_lanes<T, K>())) void k_gs(Sell A, GsDev<T> J, const T *__restrict__ g,
                                                                   double *__restrict__ dot,
                                                                   const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>();
  const int stop = stop_flag(done);
  const GsSlice S = gs_slice(J, blockIdx.x);
  const int64_t begin = A.sptr[S.s], end = FIRST ? A.smid[S.s] : A.sptr[S.s + 1];
  keep(begin, end);
  if (stop) return;
  const int64_t r = S.s * 64 + threadIdx.x / LPR;
  double prod[K / LPR] = {};
  if (r >= S.r0 && r < S.r1) gs_row<T, K, FIRST>(A, begin, end, r, r, r, T(1), threadIdx.x % LPR, g, J.x, prod);
  if (!FIRST && dot) slice_sum_store<K, LPR>(prod, dot + (int64_t)blockIdx.x * K);
}

// The merged cycles' colour: k_gs's blocks, then those of D's rows [d0, d1) in
// the same launch.  Bound by the matrix and the gathers of the other colours'
// rows, so one sweep for both cycles halves it: with it, the residual and the
// prolongation merged and the coarse levels paired, solves went from 39.2 to
// 35.2 ms (549,152 unknowns) and from 293 to 256 ms (2,179,616, K = 8).
template <class T, int K, bool FIRST>
__global__ __launch_bounds__((kWave * row_lanes<T, K>())) void k_gs_merged(Sell A, MergedRows M, GsDev<T> J,
                                                                          int64_t d0, int64_t d1,
                                                                          const T *__restrict__ g,
                                                                          double *__restrict__ dot,
                                                                          const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>();
  const int stop = stop_flag(done);
  const int t = threadIdx.x / LPR, q = threadIdx.x % LPR;
  double prod[K / LPR] = {};
  if ((int64_t)blockIdx.x >= J.nbt) {
    const Sell &X = FIRST ? M.fwd : M.bwd;
    const int64_t s = d0 / 64 + blockIdx.x - J.nbt, begin = X.sptr[s], end = X.sptr[s + 1], k = s * 64 + t;
    keep(begin, end);
    if (!stop && k >= d0 && k < d1)
      gs_row<T, K, FIRST>(X, begin, end, k, M.n + k, M.drow[k], T(1), q, g, J.x, prod);
    return;
  }
  const GsSlice S = gs_slice(J, blockIdx.x);
  const int64_t begin = A.sptr[S.s], end = FIRST ? A.smid[S.s] : A.sptr[S.s + 1];
  keep(begin, end);
  if (stop) return;
  const int64_t r = S.s * 64 + t;
  if (r >= S.r0 && r < S.r1) {
    if (!FIRST && r < M.n_top)
      gs_top_row<T, K>(M.top, r, q, g, J.x, prod);
    else
      gs_row<T, K, FIRST>(A, begin, end, r, r, r, FIRST ? T(1) : T(2), q, g, J.x, prod);
  }
  if (!FIRST && dot) slice_sum_store<K, LPR>(prod, dot + (int64_t)blockIdx.x * K);
}

// The merged cycles' residual: blocks [0, nb) as k_spmv's over all rows, the
// others R's rows.  Bound like the product by the gathers, over half the
// entries: 60 us against 95 at 2,179,616 unknowns, 148 against 251 at K = 8.
template <class T, int K>
__global__ __launch_bounds__((kBlock * row_lanes<T, K>())) void k_res_merged(Sell A, MergedRows M, int64_t nb,
                                                                            const SliceRef *__restrict__ order,
                                                                            const T *__restrict__ x,
                                                                            T *__restrict__ y,
                                                                            const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>();
  const int stop = stop_flag(done);
  const int rloc = threadIdx.x / LPR, q = threadIdx.x % LPR, w = __builtin_amdgcn_readfirstlane(rloc >> 6);
  if ((int64_t)blockIdx.x >= nb) {
    const int64_t s = (blockIdx.x - nb) * kSlicesPerBlock + w, k = s * 64 + (rloc & 63);
    if (s * 64 >= M.nr) return;
    const int64_t begin = M.res.sptr[s], end = M.res.sptr[s + 1];
    keep(begin, end);
    if (!stop && k < M.nr) residual_row<T, K>(M.res, begin, end, k, M.n + M.rpos[k], q, x, y);
    return;
  }
  const int64_t i = xcd_block(blockIdx.x, nb) * kSlicesPerBlock + w;
  if (i * 64 >= M.n) return;
  const SliceRef S = order[i];
  keep(S.end);
  if (stop) return;
  const int64_t r = S.slice * 64 + (rloc & 63);
  if (r < M.n) residual_row<T, K>(A, S.mid, S.end, r, r, q, x, y);
}

// Between the merged sweeps (MergedRows), row_lanes<T, K>() lanes per row: one
// pass in place of the two prolongations and of the sum of the two cycles.
// Bound by the vector, read and written once: 61 us at 2,179,616 unknowns, 143
// at K = 8 (a copy of it takes 57).
template <class T, int K>
__global__ __launch_bounds__((kBlock * row_lanes<T, K>())) void k_prolong_merged(MergedRows M, int64_t nb,
                                                                                const T *__restrict__ ys,
                                                                                const T *__restrict__ ya, T *x,
                                                                                const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  const int stop = stop_flag(done);
  const int rloc = threadIdx.x / LPR, q = threadIdx.x % LPR;
  const int64_t s = xcd_block(blockIdx.x, nb) * kSlicesPerBlock + __builtin_amdgcn_readfirstlane(rloc >> 6);
  const int64_t r = s * 64 + (rloc & 63);
  if (s * 64 >= M.n) return;
  const int64_t base = M.prol.sptr[s], end = M.prol.sptr[s + 1];
  keep(base, end);
  if (stop || r >= M.n) return;
  const int len = (int)((end - base) >> 6);
  const int32_t *__restrict__ cp = M.prol.col + base + (r & 63);
  const T *__restrict__ vp = sell_vals<T>(M.prol) + base + (r & 63);
  const int32_t pos = M.xpos[r];
  const Row<T, C> xr = ldp<T, K, C>(x, r, q);
  const int32_t nt = (int32_t)M.n_top;
  T es[C], pa[C];
#pragma unroll
  for (int k = 0; k < C; ++k) es[k] = pa[k] = T(0);
  auto row = [&](int32_t c) { return ldp<T, K, C>(c < nt ? ys : ya, c < nt ? c : c - nt, q); };
  auto add = [&](int32_t c, T v, const Row<T, C> &yc) {
#pragma unroll
    for (int k = 0; k < C; ++k) {
      es[k] += (c < nt ? v : T(0)) * yc.v[k];
      pa[k] += (c < nt ? T(0) : v) * yc.v[k];
    }
  };
  if constexpr (LPR == 1) {
#pragma unroll 4
    for (int e = 0; e < len; ++e) {
      const int32_t c = cp[(int64_t)e * 64];
      add(c, vp[(int64_t)e * 64], row(c));
    }
  } else {  // as sell_span
    constexpr int U = 4, N = U / LPR;
    int32_t c[N];
    T v[N];
    auto load = [&](int e0) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int e = e0 + i * LPR + q;
        c[i] = e < len ? cp[(int64_t)e * 64] : 0;
        v[i] = e < len ? vp[(int64_t)e * 64] : T(0);
      }
    };
    load(0);
    for (int e0 = 0; e0 < len; e0 += U) {
      int32_t cu[U];
      T vu[U];
      spread<LPR>(c, v, cu, vu);
      load(e0 + U);
      Row<T, C> yc[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e0 + u < len) yc[u] = row(cu[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e0 + u < len) add(cu[u], vu[u], yc[u]);
    }
  }
  Row<T, C> out;
  if (r < nt) {
#pragma unroll
    for (int k = 0; k < C; ++k) out.v[k] = xr.v[k] + es[k];
  } else {
    Row<T, C> u = xr;
    if (pos >= 0 && pos < M.nd) u = ldp<T, K, C>(x, M.n + pos, q);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      u.v[k] += pa[k];
      out.v[k] = (xr.v[k] + es[k]) + u.v[k];
    }
    if (pos >= 0) stp<T, K, C>(x, M.n + pos, q, u);
  }
  stp<T, K, C>(x, r, q, out);
}

template <class T, int K, bool ACC>
__global__ __launch_bounds__(kBlock) void k_rect(Sell E, int64_t nb, const T *__restrict__ x, T *__restrict__ y,
                                                 const int *__restrict__ done) {
  if (done && *done) return;
  const int64_t blk = xcd_block(blockIdx.x, nb);
  const int lane = threadIdx.x & 63;
  const int64_t s = blk * kSlicesPerBlock + (threadIdx.x >> 6);
  const int64_t r = s * 64 + lane;
  if (r >= E.nrows) return;
  Row<T, K> zero;
#pragma unroll
  for (int k = 0; k < K; ++k) zero.v[k] = T(0);
  T acc[K];
  sell_span<T, K, K, false>(E, E.sptr[s], E.sptr[s + 1], lane, 0, x, zero, acc);
  Row<T, K> out;
  if (ACC) out = ld<T, K>(y, r);
#pragma unroll
  for (int k = 0; k < K; ++k) out.v[k] = ACC ? out.v[k] + acc[k] : acc[k];
  st<T, K>(y, r, out);
}

template <class T, int K>
__global__ __launch_bounds__(kBlock) void k_prolong_sum(Sell E, int64_t n_top, int64_t nb, const T *__restrict__ ys,
                                                        const T *__restrict__ w, const T *__restrict__ rv,
                                                        T *__restrict__ z, double *__restrict__ partial,
                                                        const int *__restrict__ done) {
  if (done && *done) return;
  const int64_t blk = xcd_block(blockIdx.x, nb);
  const int lane = threadIdx.x & 63;
  const int64_t s = blk * kSlicesPerBlock + (threadIdx.x >> 6);
  const int64_t r = s * 64 + lane;
  double prod[K];
#pragma unroll
  for (int k = 0; k < K; ++k) prod[k] = 0.0;
  if (r < E.nrows) {
    Row<T, K> zero;
#pragma unroll
    for (int k = 0; k < K; ++k) zero.v[k] = T(0);
    T acc[K];
    sell_span<T, K, K, false>(E, E.sptr[s], E.sptr[s + 1], lane, 0, ys, zero, acc);
    Row<T, K> out;
    if (r >= n_top) {
      const Row<T, K> wr = ld<T, K>(w, r);
#pragma unroll
      for (int k = 0; k < K; ++k) out.v[k] = acc[k] + wr.v[k];
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) out.v[k] = acc[k];
    }
    st<T, K>(z, r, out);
    const Row<T, K> rr = ld<T, K>(rv, r);
#pragma unroll
    for (int k = 0; k < K; ++k) prod[k] = (double)rr.v[k] * (double)out.v[k];
  }
  block_sum_store<K>(prod, partial + blk * K);
}

// ------------------------------------------------------------- CsrG
// Up to two jobs of one launch: blocks [0, nb0) are job 0's, the rest job 1's.
template <class J>
struct Jobs {
  J j[2];
  int64_t nb0, nb1;
};

// Sums over the G groups of LPR lanes each (lane = group * LPR + q): the
// same tree over the groups whatever LPR is.
template <class T, int C, int G, int LPR>
__device__ __forceinline__ void groups_sum(T (&acc)[C]) {
  if constexpr (G > 1) {
#pragma unroll
    for (int k = 0; k < C; ++k) acc[k] = add_xor<G / 2 * LPR>(acc[k]);
    groups_sum<T, C, G / 2, LPR>(acc);
  }
}

// Entries of a row taken by one group of lanes: those t = ge, ge + G, ... of
// the n entries from b, skipping the gap [gap, gap + skip) of their storage;
// acc += v x for the C columns of lane q.  U entries are in flight at once:
// the loads past the row's end repeat its last entry and count as zero.
struct EntryRange {
  int32_t b, n, gap, skip;
};
template <class T, int C>
constexpr int entries_ahead() {
  return sizeof(T) * C > 8 ? 4 : 8;
}
template <class T, int U, int G>
__device__ __forceinline__ void load_entries(const int32_t *__restrict__ col, const T *__restrict__ val,
                                             const EntryRange &R, int32_t t0, int32_t (&c)[U], T (&v)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t t = t0 + G * u < R.n ? t0 + G * u : R.n - 1;
    const int32_t j = R.b + t + (t >= R.gap ? R.skip : 0);
    c[u] = col[j];
    v[u] = val[j];
  }
}
// x(c): the row of column c
template <class T, int C, int U, int G, class X>
__device__ __forceinline__ void add_entries(const EntryRange &R, int32_t t0, X &&x, const int32_t (&c)[U],
                                            const T (&v)[U], T (&acc)[C]) {
  Row<T, C> xc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) xc[u] = x(c[u]);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool in = t0 + G * u < R.n;
#pragma unroll
    for (int k = 0; k < C; ++k) acc[k] += v[u] * (in ? xc[u].v[k] : T(0));
  }
}
template <class T, int C, int G, int U, class X>
__device__ __forceinline__ void group_entries(const int32_t *__restrict__ col, const T *__restrict__ val,
                                              const EntryRange &R, int32_t t0, X &&x, T (&acc)[C]) {
  for (; t0 < R.n; t0 += G * U) {
    int32_t c[U];
    T v[U];
    load_entries<T, U, G>(col, val, R, t0, c, v);
    add_entries<T, C, U, G>(R, t0, x, c, v, acc);
  }
}

// A CsrG operation on row r, entries [b, e), by its G * row_lanes<T, K>() lanes.
// Bound by the chain row pointer -> entries -> gathered values at K = 1 and by
// the gathers at K = 8, where a lane of 16 bytes each makes a wavefront's load
// touch a quarter of the lines that a lane of a whole row does: with this split
// in the restrictions, residuals and sweeps, solves of 2,179,616 unknowns went
// from 106.4 to 98.6 ms and at K = 8 from 256 to 242.5.
template <class T, int K, int G, CsrMode MODE>
__device__ __forceinline__ void csr_row(const CsrG &A, int64_t r, int32_t b, int32_t e, const T *__restrict__ x,
                                        T *y) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR;
  const int l = threadIdx.x % (G * LPR), ge = l / LPR, q = l % LPR;
  // output row of a rectangular operator (its stored rows may be permuted)
  const int64_t ro = MODE != kCsrUpper && A.orow ? (int64_t)A.orow[r] : r;
  T s = T(1);
  if constexpr (MODE == kCsrUpper && !std::is_same<T, double>::value) s = A.s32[r];
  Row<T, C> out{};
  if constexpr (MODE == kCsrAdd) out = ldp<T, K, C>(y, ro, q);
  T acc[C];
#pragma unroll
  for (int k = 0; k < C; ++k) acc[k] = T(0);
  // the restrictions' rows hold about 72 entries for sixteen groups
  constexpr int U = entries_ahead<T, C>() + (sizeof(T) * C > 8 ? 1 : 0);
  group_entries<T, C, G, U>(A.col, csr_vals<T>(A), EntryRange{b, e - b, e - b, 0}, ge,
                            [&](int32_t c) { return ldp<T, K, C>(x, c, q); }, acc);
  groups_sum<T, C, G, LPR>(acc);
  if (ge != 0) return;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    if constexpr (MODE == kCsrUpper)
      out.v[k] = -s * acc[k];
    else
      out.v[k] += acc[k];
  }
  stp<T, K, C>(y, ro, q, out);
}

// The blocks of each job are renumbered like the fine kernels', so that each
// XCD works on a contiguous range of rows and the vector values those rows
// gather stay in that XCD's L2.
template <class T, int K, CsrMode MODE>
__global__ __launch_bounds__(kBlock) void k_csr(Jobs<CsrJob<T>> P, const int *__restrict__ done) {
  const int stop = stop_flag(done);
  const bool second = (int64_t)blockIdx.x >= P.nb0;
  const CsrJob<T> &J = second ? P.j[1] : P.j[0];
  const int64_t blk = second ? xcd_block(blockIdx.x - P.nb0, P.nb1) : xcd_block(blockIdx.x, P.nb0);
  const int64_t r = (blk * kBlock + threadIdx.x) / (J.A.G * row_lanes<T, K>());
  if (r >= J.A.nrows) return;
  const int32_t b = MODE == kCsrUpper ? J.A.upper[r] : J.A.ptr[r], e = J.A.ptr[r + 1];
  keep(b, e);
  if (stop) return;
  switch (J.A.G) {
    case 2: csr_row<T, K, 2, MODE>(J.A, r, b, e, J.x, J.y); break;
    case 4: csr_row<T, K, 4, MODE>(J.A, r, b, e, J.x, J.y); break;
    case 8: csr_row<T, K, 8, MODE>(J.A, r, b, e, J.x, J.y); break;
    default: csr_row<T, K, 16, MODE>(J.A, r, b, e, J.x, J.y); break;
  }
}

// Patch sweep: one block of sixteen wavefronts per patch.  First every unknown
// of the patch sums the couplings whose values the sweep takes as they stand
// (PatchRow) -- other patches (from zero only those swept before) and, with a
// start, its own patch's later unknowns (earlier ones backward) -- into
// h = g - sum (FP32: g / a_ii - sum over row-scaled values), eight groups of
// lanes an unknown.  Then the patch's factor times h, on the matrix cores:
// two wavefronts per 16 rows, each taking every second tile of the tile row,
// whose operands come straight from memory (each is used once).  No sequential
// stages inside the patch.
//
// The patch colours follow one another inside the launch.  A block takes the
// next patch in colour order (an atomic ticket), reads everything that does
// not depend on the sweep, waits until the patches of earlier colours that it
// is coupled to are done, and marks its own when its values have reached
// memory.  It waits for patches with smaller tickets only, whose blocks have
// all begun, so the earliest unfinished one never waits and every wait ends,
// whatever the order and the number in which blocks are placed.  The unknowns'
// values pass between blocks with loads and stores at agent scope, beyond the
// caches of one XCD; so each row of the halo is read once, into LDS.  Marks are
// launch numbers, which the ticket gives, so nothing is cleared in between.
// A launch per colour took 9.3 us at 129 x 129 x 33 (75 blocks a colour), of
// which the descriptors, entries and factors, now read ahead, and the launch
// were the larger part: a sweep of seven colours took 65 us in seven launches,
// 44 in one with every entry gathered at agent scope, 39 with the halo in LDS
// and a counter per colour, and takes 35 with a mark per patch (on 2,179,616
// unknowns 92, 82, 79 and 59 us, and at K = 8 113 to 150 and 85 to 102 with the
// last two).  One block a CU: two, with the factor and the entries read after
// the wait to fit their registers, took 173 us there instead of 79.
constexpr int kPatchGroups = 8;
constexpr int kPatchThreads = 1024;

template <class T>
__device__ __forceinline__ const T *patch_factor(const PatchSweep &S, bool bwd);
template <>
__device__ __forceinline__ const double *patch_factor<double>(const PatchSweep &S, bool bwd) {
  return bwd ? S.tb64 : S.tf64;
}
template <>
__device__ __forceinline__ const float *patch_factor<float>(const PatchSweep &S, bool bwd) {
  return bwd ? S.tb32 : S.tf32;
}
typedef double Tile64 __attribute__((ext_vector_type(4)));
typedef float Tile32 __attribute__((ext_vector_type(4)));
typedef unsigned Word64 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Tile64 tile_mac(double a, double b, Tile64 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Tile32 tile_mac(float a, float b, Tile32 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// row of result register r in lane l
template <class T>
__device__ __forceinline__ int tile_row(int l, int r) {
  return sizeof(T) == 8 ? l / 16 + 4 * r : 4 * (l / 16) + r;
}

// columns [q C, q C + C) of row r of a vector that other blocks of the launch
// write
template <class T, int K, int C>
__device__ __forceinline__ Row<T, C> agent_row(__amdgpu_buffer_rsrc_t x, int32_t r, int q) {
  // up to 4 GB: the offset is unsigned
  const int off = (int)(((unsigned)r * K + q * C) * (unsigned)sizeof(T));
  if constexpr (sizeof(Row<T, C>) == 4)
    return __builtin_bit_cast(Row<T, C>, __builtin_amdgcn_raw_buffer_load_b32(x, off, 0, kAgentScope));
  else if constexpr (sizeof(Row<T, C>) == 8)
    return __builtin_bit_cast(Row<T, C>, __builtin_amdgcn_raw_buffer_load_b64(x, off, 0, kAgentScope));
  else
    return __builtin_bit_cast(Row<T, C>, __builtin_amdgcn_raw_buffer_load_b128(x, off, 0, kAgentScope));
}

// FIRST: from x = 0 (forward only)
template <class T, int K, bool FIRST, bool BWD>
__global__ __launch_bounds__(kPatchThreads, 4) void k_patch_gs(Jobs<PatchJob<T>> P, const int *__restrict__ done) {
  constexpr int LPR = row_lanes<T, K>(), C = K / LPR, G = kPatchGroups, W = kPatchTile;
  constexpr int RP = kPatchThreads / (G * LPR);  // unknowns summed at once
  constexpr int NP = kPatchLdsRows / RP, U = NP == 4 ? 2 : entries_ahead<T, C>();
  using Tile = typename std::conditional<sizeof(T) == 8, Tile64, Tile32>::type;
  __shared__ Row<T, K> xs[kPatchLdsRows + kPatchHalo];  // the patch's own old values, and its halo's
  __shared__ Row<T, K> hs[kPatchLdsRows];
  __shared__ T half[kPatchLdsRows][K];
  __shared__ unsigned long long ticket;
  if (*(done ? done : &kNeverDone)) return;  // before a ticket is taken
  // the blocks of two jobs alternate while both last
  const int64_t b = blockIdx.x, both = 2 * (P.nb0 < P.nb1 ? P.nb0 : P.nb1);
  const bool second = b < both ? (b & 1) : P.nb1 > P.nb0;
  const PatchJob<T> &J = second ? P.j[1] : P.j[0];
  if (threadIdx.x == 0)
    ticket = __hip_atomic_fetch_add(J.begun, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const unsigned long long tk = ticket, launch = tk / (unsigned long long)J.np;
  const unsigned mark = __builtin_amdgcn_readfirstlane((unsigned)launch + 1);
  const int64_t pf = __builtin_amdgcn_readfirstlane((int)(tk - launch * (unsigned long long)J.np));
  const int64_t p = BWD ? J.np - 1 - pf : pf;
  const PatchDesc D = J.S.desc[p];
  const CsrG &A = J.A;
  const T *__restrict__ g = J.g, *__restrict__ vals = csr_vals<T>(A);
  const int l = threadIdx.x % (G * LPR), ge = l / LPR, q = l % LPR;
  const int m = D.m, nt = (m + W - 1) / W;
  // this wavefront's tiles: tile row I, tiles J0, J0 + 2, ...
  const int lane = threadIdx.x & 63, I = threadIdx.x >> 7, odd = (threadIdx.x >> 6) & 1;
  const int J0 = (BWD ? I : 0) + odd, J1 = I >= nt ? 0 : BWD ? nt : I + 1;
  const T *__restrict__ f = patch_factor<T>(J.S, BWD) + D.toff + lane +
                            (int64_t)((BWD ? I * nt - I * (I - 1) / 2 - I : I * (I + 1) / 2) + J0) * (W * W);
  constexpr int NT = kPatchLdsRows / W / 2;
  T a[NT][4];
  auto load_factor = [&]() {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) a[t][s] = J0 + 2 * t < J1 ? f[t * 2 * W * W + s * 64] : T(0);
  };
  // ahead of the wait unless the entries take the registers
  constexpr bool kFactorAhead = NP < 4;
  if constexpr (kFactorAhead) load_factor();
  // the staged rows: with a start the patch's own, then the halo (from zero its
  // earlier patches)
  constexpr int own = FIRST ? 0 : kPatchLdsRows;
  const int nh = FIRST ? D.nearly : D.nhalo;
  const int st = threadIdx.x / LPR, sq = threadIdx.x % LPR;
  constexpr int SP = kPatchThreads / LPR;  // rows staged at once
  auto staged = [&](int i) {  // global row of staged row i, -1: none
    return i < own ? (i < m ? D.row0 + i : -1) : i - own < nh ? J.S.halo[D.halo + i - own] : -1;
  };
  int32_t first[2];  // most patches need no more
#pragma unroll
  for (int s = 0; s < 2; ++s) first[s] = staged(st + s * SP);
  // the rows' ranges, right-hand sides and first entries
  EntryRange R[NP];
  Row<T, C> gr[NP];
  int32_t c[NP][U];
  T v[NP][U], inv[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int row = s * RP + threadIdx.x / (G * LPR);
    R[s] = EntryRange{0, 0, 0, 0};
    inv[s] = T(1);
    if (row < m) {
      const PatchRow *pr = J.S.rows + p * (kPatchLdsRows + 1) + row;
      const PatchRow r = pr[0];
      const int32_t end = pr[1].b;
      // what is taken: earlier patches; those and later ones beside the own patch's old values
      const int32_t cut = BWD ? r.late : r.own, from = BWD ? r.next : r.late;
      R[s] = EntryRange{r.b, FIRST ? r.own - r.b : cut - r.b + end - from, cut - r.b, from - cut};
      gr[s] = ldp<T, K, C>(g, D.row0 + row, q);
      if constexpr (sizeof(T) == 4) inv[s] = 1.0f / A.s32[D.row0 + row];
      if (ge < R[s].n) load_entries<T, U, G>(J.S.lcol, vals, R[s], ge, c[s], v[s]);
    }
  }
  // the coupled patches swept before this one are done
  if (threadIdx.x < kWave) {
    const int32_t n0 = BWD ? D.nbr_early : 0, n1 = BWD ? D.nbr_all : D.nbr_early;
    for (int32_t i = n0 + threadIdx.x; i < n1; i += kWave) {
      const unsigned *e = J.ended + J.S.nbr[D.nbr + i];
      while (__hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != mark) __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  const __amdgpu_buffer_rsrc_t x =
      __builtin_amdgcn_make_buffer_rsrc((void *)J.x, 0, (int)(unsigned)(A.nrows * K * sizeof(T)), 0x00027000);
  auto stage = [&](int i, int32_t r) {
    if (r >= 0)
      *reinterpret_cast<Row<T, C> *>(&xs[i < own ? i : i - own + kPatchLdsRows].v[sq * C]) = agent_row<T, K, C>(x, r, sq);
  };
#pragma unroll
  for (int s = 0; s < 2; ++s) stage(st + s * SP, first[s]);
  for (int i = st + 2 * SP; i < own + nh; i += SP) stage(i, staged(i));
  if constexpr (!kFactorAhead) load_factor();
  __syncthreads();
  auto value = [&](int32_t j) {
    return j >= 0 ? *reinterpret_cast<const Row<T, C> *>(&xs[j].v[q * C]) : agent_row<T, K, C>(x, ~j, q);
  };
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int row = s * RP + threadIdx.x / (G * LPR);
    Row<T, C> h{};
    if (row < m) {
      T acc[C];
#pragma unroll
      for (int k = 0; k < C; ++k) acc[k] = T(0);
      if (ge < R[s].n) add_entries<T, C, U, G>(R[s], ge, value, c[s], v[s], acc);
      group_entries<T, C, G, entries_ahead<T, C>()>(J.S.lcol, vals, R[s], ge + G * U, value, acc);
      groups_sum<T, C, G, LPR>(acc);
#pragma unroll
      for (int k = 0; k < C; ++k) h.v[k] = gr[s].v[k] * inv[s] - acc[k];
    }
    if (ge == 0) *reinterpret_cast<Row<T, C> *>(&hs[row].v[q * C]) = h;  // zero beyond the patch
  }
  __syncthreads();
  const int col = lane % W;
  Tile acc = {0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (J0 + 2 * t >= J1) continue;  // uniform over the wavefront
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const T bv = col < K ? hs[(J0 + 2 * t) * W + 4 * s + lane / W].v[col < K ? col : 0] : T(0);
      acc = tile_mac(a[t][s], bv, acc);
    }
  }
  if (odd && col < K) {
#pragma unroll
    for (int r = 0; r < 4; ++r) half[I * W + tile_row<T>(lane, r)][col] = acc[r];
  }
  __syncthreads();
  if (!odd && col < K) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = I * W + tile_row<T>(lane, r);
      if (row < m) {
        const T out = acc[r] + half[row][col];
        const int off = (int)(((unsigned)(D.row0 + row) * K + col) * (unsigned)sizeof(T));
        if constexpr (sizeof(T) == 8)
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Word64, out), x, off, 0, kAgentScope);
        else
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, out), x, off, 0, kAgentScope);
      }
    }
  }
  // every wavefront's values have reached memory before the patch is marked
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(J.ended + p, mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Dense FP64 coarsest inverse applied to K columns, x = C g.  C is symmetric,
// so it is read by columns (C_ji = C_ij): the 64 lanes of a wavefront take 64
// consecutive outputs i and read 64 consecutive entries of row j of C
// together, and g_j is the same for the whole wavefront; C is streamed once,
// with several rows in flight per lane.  The columns j are cut into chunks of
// kDenseChunk (dense_chunks of them); a block of kDenseWaves wavefronts takes
// 64 outputs over one chunk, each wavefront an equal part of it, sums the
// parts in LDS in wavefront order and writes the chunk's partial sums, which
// k_dense_sum adds in chunk order (a single chunk is written directly).  No
// summation order depends on K.
// Bandwidth bounds it from about 5000 unknowns (494 MB in 98 us at 6218 and
// 4820), below it the chain of loads of a wavefront, so 16 of them share a
// chunk: against four, mixed batches of eight went from 17.6 to 15.4 ms (2172
// and 2144 unknowns) and from 108.4 to 104.0 ms (2993 and 2296), with 6218 and
// 4820 unknowns unchanged.  Chunks of 128 with four wavefronts: 16.4 and 106.3.
constexpr int kDenseWaves = 16;
template <class T, int K>
__global__ __launch_bounds__(kWave *kDenseWaves) void k_dense_part(Jobs<DenseJob<T>> P,
                                                                   const int *__restrict__ done) {
  if (done && *done) return;
  const bool second = (int64_t)blockIdx.x >= P.nb0;
  const DenseJob<T> &J = second ? P.j[1] : P.j[0];
  const double *__restrict__ C = J.C;
  const int64_t m = J.m, blk = blockIdx.x - (second ? P.nb0 : 0), tiles = (m + kWave - 1) / kWave;
  __shared__ double red[kDenseWaves][K][kWave];
  __shared__ Row<T, K> gt[kDenseChunk];  // the chunk's g, read by every lane of a wavefront at once
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = blk % tiles * kWave + lane;
  const int64_t c = blk / tiles;
  const int64_t jc = c * kDenseChunk;
  const int nj = (int)(m - jc < kDenseChunk ? m - jc : kDenseChunk);
  for (int j = threadIdx.x; j < nj; j += kWave * kDenseWaves) gt[j] = ld<T, K>(J.g, jc + j);
  __syncthreads();
  constexpr int Q = kDenseChunk / kDenseWaves;
  const int j0 = w * Q;
  const int j1 = j0 + Q < nj ? j0 + Q : nj;
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  if (i < m) {
    const double *__restrict__ Ci = C + jc * m + i;
#pragma unroll 8
    for (int j = j0; j < j1; ++j) {
      const double cji = Ci[(int64_t)j * m];
      const Row<T, K> gj = gt[j];
#pragma unroll
      for (int k = 0; k < K; ++k) t[k] += cji * (double)gj.v[k];
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) red[w][k][lane] = t[k];
  __syncthreads();
  // wavefront k sums column k (K <= kDenseWaves)
  if (w >= K || i >= m) return;
  double v = red[0][w][lane];
#pragma unroll
  for (int q = 1; q < kDenseWaves; ++q) v += red[q][w][lane];
  if (m <= kDenseChunk)
    J.x[i * K + w] = (T)v;
  else
    J.part[(c * m + i) * K + w] = v;
}

template <class T, int K>
__global__ __launch_bounds__(kBlock) void k_dense_sum(Jobs<DenseJob<T>> P, const int *__restrict__ done) {
  if (done && *done) return;
  const bool second = (int64_t)blockIdx.x >= P.nb0;
  const DenseJob<T> &J = second ? P.j[1] : P.j[0];
  const int64_t t = (blockIdx.x - (second ? P.nb0 : 0)) * kBlock + threadIdx.x;  // output t = i K + k
  const int64_t m = J.m, nc = (m + kDenseChunk - 1) / kDenseChunk;
  if (t >= m * K) return;
  double s = J.part[t];
#pragma unroll 8
  for (int64_t c = 1; c < nc; ++c) s += J.part[c * m * K + t];
  J.x[t] = (T)s;
}

// ------------------------------------------------------------- vectors
template <class T>
__global__ void k_fill(T *__restrict__ x, int64_t n, T v, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

template <class T>
__global__ void k_copy(const T *__restrict__ a, T *__restrict__ b, int64_t n, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}

template <class T, int K>
__global__ __launch_bounds__(kBlock) void k_dot(const T *__restrict__ a, const T *__restrict__ b, int64_t n,
                                                double *__restrict__ partial, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  if (i < n) {
    const Row<T, K> ai = ld<T, K>(a, i), bi = ld<T, K>(b, i);
#pragma unroll
    for (int k = 0; k < K; ++k) t[k] = (double)ai.v[k] * (double)bi.v[k];
  }
  block_sum_store<K>(t, partial + (int64_t)blockIdx.x * K);
}

// z_i += w_i on the rows i >= row0, then the block partials of r . z
template <class T, int K>
__global__ __launch_bounds__(kBlock) void k_add_dot(const T *__restrict__ w, const T *__restrict__ r,
                                                    T *__restrict__ z, int64_t row0, int64_t n,
                                                    double *__restrict__ partial, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  if (i < n) {
    Row<T, K> zi = ld<T, K>(z, i);
    const Row<T, K> ri = ld<T, K>(r, i);
    if (i >= row0) {
      const Row<T, K> wi = ld<T, K>(w, i);
#pragma unroll
      for (int k = 0; k < K; ++k) zi.v[k] += wi.v[k];
      st<T, K>(z, i, zi);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) t[k] = (double)ri.v[k] * (double)zi.v[k];
  }
  block_sum_store<K>(t, partial + (int64_t)blockIdx.x * K);
}

template <class T, int K>
__global__ void k_jacobi(const T *__restrict__ r, const double *__restrict__ dg, T *__restrict__ z, int64_t n,
                         const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Row<T, K> ri = ld<T, K>(r, i);
  Row<T, K> out;
  const double d = dg[i];
#pragma unroll
  for (int k = 0; k < K; ++k) out.v[k] = (T)((double)ri.v[k] / d);
  st<T, K>(z, i, out);
}

__global__ void k_gather(const double *__restrict__ nat, const int64_t *__restrict__ perm, double *__restrict__ sto,
                         int64_t n, int K, int k) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) sto[i * K + k] = nat[perm[i]];
}

__global__ void k_scatter(const double *__restrict__ sto, const int64_t *__restrict__ perm, double *__restrict__ nat,
                          int64_t n, int K, int k) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) nat[perm[i]] = sto[i * K + k];
}

// all columns of a batch at once, a thread per row: whole rows are written or
// read (a launch per column touched every line of the batch's vector each time:
// a mixed solve of three columns on 10,625 nodes, 5.57 ms, took 5.49 with this)
template <int K>
__global__ void k_gather_batch(const double *__restrict__ nat, int64_t N, const int64_t *__restrict__ perm,
                               double *__restrict__ sto, int64_t n, int cols) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t p = perm[i];
  Row<double, K> v{};
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (k < cols) v.v[k] = nat[k * N + p];
  st<double, K>(sto, i, v);
}

template <int K>
__global__ void k_scatter_batch(const double *__restrict__ sto, const int32_t *__restrict__ pos,
                                double *__restrict__ nat, int64_t N, int cols) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int32_t p = pos[i];
  Row<double, K> v{};
  if (p >= 0) v = ld<double, K>(sto, p);
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (k < cols) nat[k * N + i] = v.v[k];
}

__global__ void k_demote(const double *__restrict__ r64, const double *__restrict__ scale, float *__restrict__ r32,
                         int64_t n, int K, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * K) r32[i] = (float)(r64[i] * scale[i % K]);
}

__global__ void k_promote(const float *__restrict__ d32, const double *__restrict__ scale, double *__restrict__ x64,
                          int64_t n, int K, const int *__restrict__ done) {
  if (done && *done) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * K) return;
  x64[i] = scale[i % K] * (double)d32[i];
}

// ------------------------------------------------------------- PCG scalars
// Fixed-order sums of the K columns of np partials (row-major [np][K]) by one
// block, all columns at once: thread t adds rows t, t + kBlock, ... in turn,
// then a pairwise tree over the threads.  The order for column k does not
// depend on K, so a column's sum is the same alone and in a batch.
__device__ __forceinline__ void sum_partials(const double *__restrict__ p, int64_t np, int K,
                                             double (&res)[kMaxBatch]) {
  double t[kMaxBatch];
#pragma unroll
  for (int k = 0; k < kMaxBatch; ++k) t[k] = 0.0;
  // eight of each thread's partials are loaded before any is added, so that
  // a thread keeps eight loads per column in flight; the additions keep the
  // order j = tid, tid + kBlock, ...
  constexpr int U = 8;
  int64_t j = threadIdx.x;
  for (; j + (U - 1) * kBlock < np; j += U * kBlock) {
    double v[U][kMaxBatch];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < kMaxBatch; ++k) v[u][k] = (k < K) ? p[(j + u * kBlock) * K + k] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < kMaxBatch; ++k)
        if (k < K) t[k] += v[u][k];
  }
  for (; j < np; j += kBlock) {
#pragma unroll
    for (int k = 0; k < kMaxBatch; ++k)
      if (k < K) t[k] += p[j * K + k];
  }
  // then a fixed tree: xor shuffles within each wavefront, and the four
  // wavefront sums added in order (the same result in every thread)
  __shared__ double buf[kMaxBatch][kSlicesPerBlock];
#pragma unroll
  for (int k = 0; k < kMaxBatch; ++k)
    if (k < K) t[k] = wave_sum(t[k]);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) {
#pragma unroll
    for (int k = 0; k < kMaxBatch; ++k)
      if (k < K) buf[k][threadIdx.x / kWave] = t[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMaxBatch; ++k) {
    double r = 0.0;
    if (k < K) {
#pragma unroll
      for (int w = 0; w < kSlicesPerBlock; ++w) r += buf[k][w];
    }
    res[k] = r;
  }
}

// Lanes that load one partial row of K columns, 16 bytes each (one lane of 8
// bytes for K = 1), and the block size of the kernels that use
// sum_partials_wide.
template <int K>
constexpr int partial_lanes() {
  return K >= 2 ? K / 2 : 1;
}
template <int K>
constexpr int wide_block() {
  return kBlock * partial_lanes<K>();
}

// sum_partials for a K known at compile time, by a block of wide_block<K>()
// threads: the lanes of row group v (partial_lanes<K>() consecutive threads)
// load rows v, v + kBlock, ... whole, one 16-byte piece each, so that a
// wavefront reads consecutive rows and keeps several times the loads in
// flight.  Each lane adds its columns over those rows in that order, which
// is thread v's order in sum_partials, and the first kBlock threads then
// take thread v's place in its tree: the result equals sum_partials' bit for
// bit.  Every thread of the block must call it.
template <int K>
__device__ __forceinline__ void sum_partials_wide(const double *__restrict__ p, int64_t np,
                                                  double (&res)[kMaxBatch]) {
  constexpr int LP = partial_lanes<K>(), CW = K / LP;
  const int v = threadIdx.x / LP, c = threadIdx.x % LP;
  double t[CW];
#pragma unroll
  for (int k = 0; k < CW; ++k) t[k] = 0.0;
  auto load = [&](int64_t j, double(&w)[CW]) {
    if constexpr (CW == 2) {
      const double2 q = *reinterpret_cast<const double2 *>(p + j * K + c * 2);
      w[0] = q.x;
      w[1] = q.y;
    } else {
      w[0] = p[j * K + c];
    }
  };
  constexpr int U = 8;
  int64_t j = v;
  for (; j + (U - 1) * kBlock < np; j += U * kBlock) {
    double w[U][CW];
#pragma unroll
    for (int u = 0; u < U; ++u) load(j + u * kBlock, w[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < CW; ++k) t[k] += w[u][k];
  }
  for (; j < np; j += kBlock) {
    double w[CW];
    load(j, w);
#pragma unroll
    for (int k = 0; k < CW; ++k) t[k] += w[k];
  }
  __shared__ double col[K][kBlock];
#pragma unroll
  for (int k = 0; k < CW; ++k) col[c * CW + k][v] = t[k];
  __syncthreads();
  __shared__ double buf[K][kSlicesPerBlock];
  if (threadIdx.x < kBlock) {  // whole wavefronts
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double w = wave_sum(col[k][threadIdx.x]);
      if ((threadIdx.x & (kWave - 1)) == 0) buf[k][threadIdx.x / kWave] = w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMaxBatch; ++k) {
    double r = 0.0;
    if (k < K) {
#pragma unroll
      for (int w = 0; w < kSlicesPerBlock; ++w) r += buf[k][w];
    }
    res[k] = r;
  }
}

__device__ __forceinline__ void update_all_done(Scal *s) {
  int all = 1;
  for (int k = 0; k < s->K; ++k) all &= s->done[k];
  s->all_done = all;
}

__global__ __launch_bounds__(kBlock) void k_reduce(const double *p, int64_t np, int K, double *out) {
  double t[kMaxBatch];
  sum_partials(p, np, K, t);
  if (threadIdx.x == 0)
    for (int k = 0; k < K; ++k) out[k] = t[k];
}

__global__ __launch_bounds__(kBlock) void k_pcg_init(Scal *s, const double *pb, int64_t npb, int K, double tol,
                                                     int maxit, double *scale_in, double *scale_out) {
  double sums[kMaxBatch];
  sum_partials(pb, npb, K, sums);
  for (int k = 0; k < kMaxBatch; ++k) {
    const double t = sums[k];
    if (threadIdx.x == 0) {
      s->bnorm2[k] = t;
      s->iters[k] = 0;
      s->rho[k] = 0.0;
      s->alpha[k] = 0.0;
      s->beta[k] = 0.0;
      if (scale_in && k < K) {
        const double nb = sqrt(t);
        const bool ok = nb > 0.0 && isfinite(nb);
        scale_in[k] = ok ? 1.0 / nb : 0.0;
        scale_out[k] = ok ? nb : 0.0;
      }
      if (k >= K || t == 0.0) {
        s->done[k] = 1;
        s->status[k] = 1;
      } else if (!isfinite(t)) {
        s->done[k] = 1;
        s->status[k] = -6;
      } else {
        s->done[k] = 0;
        s->status[k] = 0;
      }
    }
  }
  if (threadIdx.x == 0) {
    s->K = K;
    for (int k = 0; k < kMaxBatch; ++k) {
      s->tol2[k] = tol * tol;
      s->maxit[k] = maxit;
    }
    update_all_done(s);
  }
}

__global__ __launch_bounds__(kBlock) void k_pcg_set_rho(Scal *s, const double *p, int64_t np) {
  double t[kMaxBatch];
  sum_partials(p, np, s->K, t);
  if (threadIdx.x == 0)
    for (int k = 0; k < s->K; ++k) s->rho[k] = t[k];
}

// The per-iteration scalar kernels handle column k in thread k, so that the
// few loads and stores of each column overlap instead of following one
// another in a single thread.
__device__ __forceinline__ double column_of(const double (&v)[kMaxBatch], int k) {
  double out = 0.0;
#pragma unroll
  for (int q = 0; q < kMaxBatch; ++q)
    if (q == k) out = v[q];
  return out;
}

// all_done from the columns' flags (thread k < K holds column k's); every
// thread of the block must call it
__device__ __forceinline__ void store_all_done(Scal *s, int K, int mine) {
  __shared__ int flags[kMaxBatch];
  if ((int)threadIdx.x < K) flags[threadIdx.x] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    int all = 1;
    for (int k = 0; k < K; ++k) all &= flags[k];
    s->all_done = all;
  }
}

// sum_partials for a K known at compile time, by a block of kBlock threads
template <int K>
__device__ __forceinline__ void sum_rows(const double *__restrict__ p, int64_t np, double (&res)[K]) {
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  constexpr int U = K >= 4 ? 2 : 8;
  for (int64_t j = threadIdx.x; j < np; j += U * kBlock) {
    Row<double, K> w[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j + u * kBlock < np) w[u] = ld<double, K>(p, j + u * kBlock);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j + u * kBlock < np) {
#pragma unroll
        for (int k = 0; k < K; ++k) t[k] += w[u].v[k];
      }
  }
  __shared__ double buf[K][kSlicesPerBlock];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = wave_sum(t[k]);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) buf[k][threadIdx.x / kWave] = t[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kSlicesPerBlock; ++w) r += buf[k][w];
    res[k] = r;
  }
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_compact(const double *__restrict__ p, int64_t np,
                                                    double *__restrict__ out, const int *__restrict__ done) {
  const int stop = stop_flag(done);
  if (stop) return;
  const int64_t chunk = (np + kCompact - 1) / kCompact, r0 = blockIdx.x * chunk;
  double s[K];
  sum_rows<K>(p + r0 * K, r0 >= np ? 0 : np - r0 < chunk ? np - r0 : chunk, s);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) out[(int64_t)blockIdx.x * K + k] = s[k];
  }
}

// The scalar steps of one column, from the record `s` and the column's sum.
struct Alpha {
  double alpha;
  int done, status;
};
__device__ __forceinline__ Alpha alpha_step(const Scal *s, int k, double pq) {
  Alpha a{s->alpha[k], s->done[k], s->status[k]};
  if (a.done) return a;
  const double rho = s->rho[k];
  if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) return Alpha{0.0, 1, -6};
  a.alpha = rho / pq;
  return a;
}
struct Conv {
  int iters, done, status;
};
__device__ __forceinline__ Conv conv_step(const Scal *s, int k, double rr) {
  Conv c{s->iters[k], s->done[k], s->status[k]};
  if (c.done) return c;
  ++c.iters;
  c.status = !isfinite(rr) ? -6 : rr <= s->tol2[k] * s->bnorm2[k] ? 1 : c.iters >= s->maxit[k] ? 2 : 0;
  c.done = c.status != 0;
  return c;
}
// thread k copies column k's record (the columns beyond K too)
__device__ __forceinline__ void copy_record(const Scal *in, Scal *out) {
  const int k = threadIdx.x;
  if (k < kMaxBatch) {
    out->rho[k] = in->rho[k];
    out->alpha[k] = in->alpha[k];
    out->beta[k] = in->beta[k];
    out->bnorm2[k] = in->bnorm2[k];
    out->rr[k] = in->rr[k];
    out->pq[k] = in->pq[k];
    out->tol2[k] = in->tol2[k];
    out->done[k] = in->done[k];
    out->iters[k] = in->iters[k];
    out->status[k] = in->status[k];
    out->maxit[k] = in->maxit[k];
  }
  if (k == 0) {
    out->all_done = in->all_done;
    out->K = in->K;
  }
}

template <int K>
__global__ __launch_bounds__(wide_block<K>()) void k_pcg_alpha(const Scal *in, Scal *out, const double *p,
                                                               int64_t np) {
  copy_record(in, out);
  if (in->all_done) return;
  double sums[kMaxBatch];
  sum_partials_wide<K>(p, np, sums);
  const int k = threadIdx.x;
  int done = 1;
  if (k < K) {
    const double pq = column_of(sums, k);
    const Alpha a = alpha_step(in, k, pq);
    if (!in->done[k]) out->pq[k] = pq;
    out->alpha[k] = a.alpha;
    out->status[k] = a.status;
    out->done[k] = done = a.done;
  }
  store_all_done(out, K, done);
}

// FOLD: the block forms alpha itself (in -> out written by the first block);
// else `in` holds it.  Bound by its six vectors (153 to 173 us at 2,179,616
// unknowns and K = 8, the rate of a copy); small, by the launch it saves.
template <class T, int K, bool FOLD, bool DEMOTE>
__global__ __launch_bounds__(kBlock) void k_pcg_xr(const Scal *__restrict__ in, Scal *__restrict__ out,
                                                   const double *__restrict__ pq, int64_t np, T *__restrict__ x,
                                                   T *__restrict__ r, const T *__restrict__ p,
                                                   const T *__restrict__ q, int64_t n, double *__restrict__ partial,
                                                   float *__restrict__ r32, const double *__restrict__ scale) {
  if (FOLD && blockIdx.x == 0) copy_record(in, out);
  if (in->all_done) return;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  Row<T, K> xi{}, ri{}, pi{}, qi{};
  if (i < n) {
    xi = ld<T, K>(x, i);
    ri = ld<T, K>(r, i);
    pi = ld<T, K>(p, i);
    qi = ld<T, K>(q, i);
  }
  double al[K];
  int dn[K];
  if constexpr (FOLD) {
    double sums[K];
    sum_rows<K>(pq, np, sums);
    int all = 1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const Alpha a = alpha_step(in, k, sums[k]);
      al[k] = a.alpha;
      dn[k] = a.done;
      all &= a.done;
      if (blockIdx.x == 0 && threadIdx.x == k) {
        if (!in->done[k]) out->pq[k] = sums[k];
        out->alpha[k] = a.alpha;
        out->status[k] = a.status;
        out->done[k] = a.done;
      }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out->all_done = all;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      al[k] = in->alpha[k];
      dn[k] = in->done[k];
    }
  }
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  if (i < n) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!dn[k]) {
        const T a = (T)al[k];
        xi.v[k] += a * pi.v[k];
        ri.v[k] -= a * qi.v[k];
      }
      t[k] = (double)ri.v[k] * (double)ri.v[k];
    }
    st<T, K>(x, i, xi);
    st<T, K>(r, i, ri);
    if constexpr (DEMOTE) {
      Row<float, K> d;
#pragma unroll
      for (int k = 0; k < K; ++k) d.v[k] = (float)((double)ri.v[k] * scale[k]);
      st<float, K>(r32, i, d);
    }
  }
  block_sum_store<K>(t, partial + (int64_t)blockIdx.x * K);
}

template <int K>
__global__ __launch_bounds__(wide_block<K>()) void k_pcg_conv(Scal *s, const double *p, int64_t np) {
  if (s->all_done) return;
  double sums[kMaxBatch];
  sum_partials_wide<K>(p, np, sums);
  const int k = threadIdx.x;
  int done = 1;
  if (k < K) {
    const Conv c = conv_step(s, k, column_of(sums, k));
    if (!s->done[k]) s->rr[k] = column_of(sums, k);
    s->iters[k] = c.iters;
    s->status[k] = c.status;
    s->done[k] = done = c.done;
  }
  store_all_done(s, K, done);
}

template <int K>
__global__ __launch_bounds__(wide_block<K>()) void k_pcg_beta(const Scal *in, Scal *out, const double *p,
                                                              int64_t np) {
  copy_record(in, out);
  if (in->all_done) return;
  double sums[kMaxBatch];
  sum_partials_wide<K>(p, np, sums);
  const int k = threadIdx.x;
  if (k < K && !in->done[k]) {
    const double rz = column_of(sums, k);
    out->beta[k] = rz / in->rho[k];
    out->rho[k] = rz;
  }
}

// Bound by its three vectors (75 us at 2,179,616 unknowns and K = 8).
// FOLD: the block forms beta itself (in -> out written by the first block), and
// with CONV applies the convergence test; else `in` holds them.
template <class T, int K, bool FOLD, bool CONV>
__global__ __launch_bounds__(kBlock) void k_pcg_p(const Scal *__restrict__ in, Scal *__restrict__ out,
                                                  const double *__restrict__ rr, int64_t nrr,
                                                  const double *__restrict__ rz, int64_t nrz, T *__restrict__ p,
                                                  const T *__restrict__ z, int64_t n) {
  if (FOLD && blockIdx.x == 0) copy_record(in, out);
  if (in->all_done) return;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  Row<T, K> pi{}, zi{};
  if (i < n) {
    pi = ld<T, K>(p, i);
    zi = ld<T, K>(z, i);
  }
  double be[K];
  int dn[K];
  if constexpr (FOLD) {
    double s[K], sz[K];
    if constexpr (CONV) sum_rows<K>(rr, nrr, s);
    sum_rows<K>(rz, nrz, sz);
    int all = 1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      dn[k] = in->done[k];
      be[k] = sz[k] / in->rho[k];
      const bool mine = blockIdx.x == 0 && threadIdx.x == k;
      if constexpr (CONV) {
        const Conv c = conv_step(in, k, s[k]);
        if (mine) {
          if (!dn[k]) out->rr[k] = s[k];
          out->iters[k] = c.iters;
          out->status[k] = c.status;
          out->done[k] = c.done;
        }
        dn[k] = c.done;
      }
      all &= dn[k];
      if (mine && !dn[k]) {
        out->beta[k] = be[k];
        out->rho[k] = sz[k];
      }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out->all_done = all;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      be[k] = in->beta[k];
      dn[k] = in->done[k];
    }
  }
  if (i >= n) return;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (!dn[k]) pi.v[k] = zi.v[k] + (T)be[k] * pi.v[k];
  st<T, K>(p, i, pi);
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_promote_dot(const float *__restrict__ z32,
                                                        const double *__restrict__ scale,
                                                        const double *__restrict__ r, double *__restrict__ z64,
                                                        int64_t n, double *__restrict__ partial,
                                                        const int *__restrict__ done) {
  const int stop = stop_flag(done);
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) t[k] = 0.0;
  if (stop) return;
  if (i < n) {
    const Row<float, K> zi = ld<float, K>(z32, i);
    const Row<double, K> ri = ld<double, K>(r, i);
    Row<double, K> out;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      out.v[k] = scale[k] * (double)zi.v[k];
      t[k] = ri.v[k] * out.v[k];
    }
    st<double, K>(z64, i, out);
  }
  block_sum_store<K>(t, partial + (int64_t)blockIdx.x * K);
}

__global__ void k_pcg_resume(Scal *s, unsigned keep) {
  if (threadIdx.x == 0) {
    for (int k = 0; k < s->K; ++k)
      if (!((keep >> k) & 1u)) {
        s->done[k] = 0;
        s->status[k] = 0;
      }
    update_all_done(s);
  }
}

__global__ void k_slot_vectors(unsigned mask, int restart, const double *__restrict__ b, const double *__restrict__ res,
                               double *__restrict__ hi, double *__restrict__ lo, double *__restrict__ x,
                               double *__restrict__ r, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * kMaxBatch) return;
  int k = (int)(i % kMaxBatch);
  if (!((mask >> k) & 1u)) return;
  if (restart) {
    r[i] = res[i];
  } else {
    hi[i] = 0.0;
    lo[i] = 0.0;
    x[i] = 0.0;
    r[i] = b[i];
  }
}

__global__ __launch_bounds__(kBlock) void k_slot_scalars(unsigned mask, int restart, Scal *s, const double *pb,
                                                         int64_t npb, SlotStop stop, double *scale_in,
                                                         double *scale_out) {
  double sums[kMaxBatch];
  sum_partials(pb, npb, kMaxBatch, sums);
  for (int k = 0; k < kMaxBatch; ++k) {
    if (!((mask >> k) & 1u)) continue;
    const double t = restart ? 0.0 : sums[k];
    if (threadIdx.x == 0) {
      if (!restart) {
        s->bnorm2[k] = t;
        s->iters[k] = 0;
        s->tol2[k] = stop.tol[k] * stop.tol[k];
        s->maxit[k] = stop.maxit[k];
        double nb = sqrt(t);
        bool ok = t > 0.0 && isfinite(t);
        scale_in[k] = ok ? 1.0 / nb : 0.0;
        scale_out[k] = ok ? nb : 0.0;
      }
      const double bb = s->bnorm2[k];
      if (bb == 0.0) {
        s->done[k] = 1;
        s->status[k] = 1;
      } else if (!isfinite(bb)) {
        s->done[k] = 1;
        s->status[k] = -6;
      } else {
        s->done[k] = 0;
        s->status[k] = 0;
      }
    }
  }
  if (threadIdx.x == 0) {
    s->K = kMaxBatch;
    update_all_done(s);
  }
}

__global__ __launch_bounds__(kBlock) void k_slot_rho(unsigned mask, Scal *s, const double *p, int64_t np) {
  double t[kMaxBatch];
  sum_partials(p, np, kMaxBatch, t);
  if (threadIdx.x == 0)
    for (int k = 0; k < kMaxBatch; ++k)
      if ((mask >> k) & 1u) s->rho[k] = t[k];
}

__global__ void k_slot_copy(unsigned mask, const double *__restrict__ z, double *__restrict__ p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * kMaxBatch) return;
  if ((mask >> (int)(i % kMaxBatch)) & 1u) p[i] = z[i];
}

inline dim3 grid(int64_t nb) { return dim3((unsigned)nb); }

}  // namespace

void launch_slot_vectors(hipStream_t stm, unsigned mask, bool restart, const double *b, const double *res, double *hi,
                         double *lo, double *x, double *r, int64_t n) {
  if (n <= 0 || !mask) return;
  hipLaunchKernelGGL(k_slot_vectors, grid(vec_blocks(n * kMaxBatch)), dim3(kBlock), 0, stm, mask, (int)restart, b, res,
                     hi, lo, x, r, n);
}
void launch_slot_scalars(hipStream_t stm, unsigned mask, bool restart, Scal *s, const double *pb, int64_t npb,
                         const SlotStop &stop, double *scale_in, double *scale_out) {
  hipLaunchKernelGGL(k_slot_scalars, dim3(1), dim3(kBlock), 0, stm, mask, (int)restart, s, pb, npb, stop,
                     scale_in, scale_out);
}
void launch_slot_rho(hipStream_t stm, unsigned mask, Scal *s, const double *p, int64_t np) {
  hipLaunchKernelGGL(k_slot_rho, dim3(1), dim3(kBlock), 0, stm, mask, s, p, np);
}
void launch_slot_copy(hipStream_t stm, unsigned mask, const double *z, double *p, int64_t n) {
  if (n <= 0 || !mask) return;
  hipLaunchKernelGGL(k_slot_copy, grid(vec_blocks(n * kMaxBatch)), dim3(kBlock), 0, stm, mask, z, p, n);
}

#define VEMG_K_SWITCH(K, ...) \
  switch (K) {                \
    case 1: {                 \
      constexpr int KK = 1;   \
      __VA_ARGS__;            \
    } break;                  \
    case 2: {                 \
      constexpr int KK = 2;   \
      __VA_ARGS__;            \
    } break;                  \
    case 4: {                 \
      constexpr int KK = 4;   \
      __VA_ARGS__;            \
    } break;                  \
    default: {                \
      constexpr int KK = 8;   \
      __VA_ARGS__;            \
    } break;                  \
  }

template <class T>
void launch_spmv(hipStream_t stm, int K, const Sell &A, int mode, int64_t r0, int64_t r1, const T *x, T *y,
                 double *partial, const int *done, const SliceRef *order) {
  int64_t nb = sell_blocks(r0, r1);
  if (!nb) return;
  const int64_t ns = (r1 + kWave - 1) / kWave - r0 / kWave;
  VEMG_K_SWITCH(K, {
    const dim3 blk(kBlock * row_lanes<T, KK>());
    if (mode == 0) {
      if (partial)
        hipLaunchKernelGGL((k_spmv<T, KK, 0, true>), grid(nb), blk, 0, stm, A, r0, r1, ns, nb, order, x, y,
                           partial, done);
      else
        hipLaunchKernelGGL((k_spmv<T, KK, 0, false>), grid(nb), blk, 0, stm, A, r0, r1, ns, nb, order, x, y,
                           partial, done);
    } else {
      hipLaunchKernelGGL((k_spmv<T, KK, 1, false>), grid(nb), blk, 0, stm, A, r0, r1, ns, nb, order, x, y,
                         partial, done);
    }
  })
}

static inline int64_t slices(int64_t r0, int64_t r1) {
  return r1 <= r0 ? 0 : (r1 + kWave - 1) / kWave - r0 / kWave;
}

template <class T>
static GsDev<T> gs_ranges(int64_t a0, int64_t a1, int64_t b0, int64_t b1, T *x) {
  GsDev<T> J{};
  J.x = x;
  const int64_t ra[2] = {a0, b0}, rb[2] = {a1, b1};
  for (int i = 0; i < 2; ++i) {
    const int64_t nb = slices(ra[i], rb[i]);
    if (!nb) continue;
    J.r0[J.n] = ra[i];
    J.r1[J.n] = rb[i];
    J.sf[J.n] = ra[i] / kWave;
    J.nb[J.n] = nb;
    J.nbt += nb;
    ++J.n;
  }
  return J;
}

template <class T>
int64_t launch_gs(hipStream_t stm, int K, const Sell &A, int64_t a0, int64_t a1, int64_t b0, int64_t b1, const T *g,
                  T *x, const int *done, bool first, double *dot) {
  const GsDev<T> J = gs_ranges(a0, a1, b0, b1, x);
  if (!J.nbt) return 0;
  VEMG_K_SWITCH(K, {
    const dim3 blk(kWave * row_lanes<T, KK>());
    if (first)
      hipLaunchKernelGGL((k_gs<T, KK, true>), grid(J.nbt), blk, 0, stm, A, J, g, dot, done);
    else
      hipLaunchKernelGGL((k_gs<T, KK, false>), grid(J.nbt), blk, 0, stm, A, J, g, dot, done);
  })
  return J.nbt;
}

template <class T>
int64_t launch_gs_merged(hipStream_t stm, int K, const Sell &A, const MergedRows &M, int64_t a0, int64_t a1,
                         int64_t b0, int64_t b1, int64_t d0, int64_t d1, const T *g, T *x, const int *done,
                         bool first, double *dot) {
  const GsDev<T> J = gs_ranges(a0, a1, b0, b1, x);
  const int64_t nb = J.nbt + slices(d0, d1);
  if (!nb) return 0;
  VEMG_K_SWITCH(K, {
    const dim3 blk(kWave * row_lanes<T, KK>());
    if (first)
      hipLaunchKernelGGL((k_gs_merged<T, KK, true>), grid(nb), blk, 0, stm, A, M, J, d0, d1, g, dot, done);
    else
      hipLaunchKernelGGL((k_gs_merged<T, KK, false>), grid(nb), blk, 0, stm, A, M, J, d0, d1, g, dot, done);
  })
  return J.nbt;
}

template <class T>
void launch_res_merged(hipStream_t stm, int K, const Sell &A, const MergedRows &M, const T *x, T *y, const int *done,
                       const SliceRef *order) {
  const int64_t nb = sell_blocks(0, M.n), nbx = vec_blocks(M.nr);
  if (!nb) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_res_merged<T, KK>), grid(nb + nbx), dim3(kBlock * row_lanes<T, KK>()), 0,
                                      stm, A, M, nb, order, x, y, done))
}

template <class T>
void launch_prolong_merged(hipStream_t stm, int K, const MergedRows &M, const T *ys, const T *ya, T *x,
                           const int *done) {
  const int64_t nb = vec_blocks(M.n);
  if (!nb) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_prolong_merged<T, KK>), grid(nb), dim3(kBlock * row_lanes<T, KK>()), 0, stm,
                                      M, nb, ys, ya, x, done))
}

template <class T>
void launch_rect(hipStream_t stm, int K, const Sell &E, bool accumulate, const T *x, T *y, const int *done) {
  int64_t nb = sell_blocks(0, E.nrows);
  if (!nb) return;
  VEMG_K_SWITCH(K, {
    if (accumulate)
      hipLaunchKernelGGL((k_rect<T, KK, true>), grid(nb), dim3(kBlock), 0, stm, E, nb, x, y, done);
    else
      hipLaunchKernelGGL((k_rect<T, KK, false>), grid(nb), dim3(kBlock), 0, stm, E, nb, x, y, done);
  })
}

template <class T>
void launch_prolong_sum(hipStream_t stm, int K, const Sell &E, int64_t n_top, const T *y, const T *w, const T *r,
                        T *z, double *partial, const int *done) {
  int64_t nb = sell_blocks(0, E.nrows);
  if (!nb) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_prolong_sum<T, KK>), grid(nb), dim3(kBlock), 0, stm, E, n_top, nb, y, w, r,
                                      z, partial, done))
}

// the one or two jobs of a launch, blocks(job) of them each
template <class J, class F>
static Jobs<J> two_jobs(const J *jobs, int nj, F &&blocks) {
  Jobs<J> P{};
  P.j[0] = jobs[0];
  P.nb0 = blocks(jobs[0]);
  if (nj > 1) {
    P.j[1] = jobs[1];
    P.nb1 = blocks(jobs[1]);
  }
  return P;
}

template <class T>
void launch_csr(hipStream_t stm, int K, CsrMode mode, const CsrJob<T> *jobs, int nj, const int *done) {
  VEMG_K_SWITCH(K, {
    const auto P = two_jobs(jobs, nj, [](const CsrJob<T> &j) {
      return (j.A.nrows * j.A.G * row_lanes<T, KK>() + kBlock - 1) / kBlock;
    });
    const int64_t nb = P.nb0 + P.nb1;
    if (!nb) return;
    if (mode == kCsrUpper)
      hipLaunchKernelGGL((k_csr<T, KK, kCsrUpper>), grid(nb), dim3(kBlock), 0, stm, P, done);
    else if (mode == kCsrMult)
      hipLaunchKernelGGL((k_csr<T, KK, kCsrMult>), grid(nb), dim3(kBlock), 0, stm, P, done);
    else
      hipLaunchKernelGGL((k_csr<T, KK, kCsrAdd>), grid(nb), dim3(kBlock), 0, stm, P, done);
  })
}

template <class T>
void launch_patch_gs(hipStream_t stm, int K, PatchDir dir, const PatchJob<T> *jobs, int nj, const int *done) {
  const auto P = two_jobs(jobs, nj, [](const PatchJob<T> &j) { return j.np; });
  const int64_t nb = P.nb0 + P.nb1;
  if (!nb) return;
  VEMG_K_SWITCH(K, {
    if (dir == kPatchFirst)
      hipLaunchKernelGGL((k_patch_gs<T, KK, true, false>), grid(nb), dim3(kPatchThreads), 0, stm, P, done);
    else if (dir == kPatchBackward)
      hipLaunchKernelGGL((k_patch_gs<T, KK, false, true>), grid(nb), dim3(kPatchThreads), 0, stm, P, done);
    else
      hipLaunchKernelGGL((k_patch_gs<T, KK, false, false>), grid(nb), dim3(kPatchThreads), 0, stm, P, done);
  })
}

template <class T>
void launch_dense(hipStream_t stm, int K, const DenseJob<T> *jobs, int nj, const int *done) {
  const auto P = two_jobs(jobs, nj, [](const DenseJob<T> &j) {
    return (j.m + kWave - 1) / kWave * dense_chunks(j.m);
  });
  if (!(P.nb0 + P.nb1)) return;
  VEMG_K_SWITCH(K, {
    hipLaunchKernelGGL((k_dense_part<T, KK>), grid(P.nb0 + P.nb1), dim3(kWave * kDenseWaves), 0, stm, P, done);
    // a single chunk is complete already
    const auto S = two_jobs(jobs, nj, [](const DenseJob<T> &j) {
      return dense_chunks(j.m) > 1 ? (j.m * KK + kBlock - 1) / kBlock : int64_t(0);
    });
    if (S.nb0 + S.nb1)
      hipLaunchKernelGGL((k_dense_sum<T, KK>), grid(S.nb0 + S.nb1), dim3(kBlock), 0, stm, S, done);
  })
}

template <class T>
void launch_fill(hipStream_t stm, T *x, int64_t n, T v, const int *done) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_fill<T>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, x, n, v, done);
}

template <class T>
void launch_copy(hipStream_t stm, const T *a, T *b, int64_t n, const int *done) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_copy<T>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, a, b, n, done);
}

template <class T>
void launch_dot(hipStream_t stm, int K, const T *a, const T *b, int64_t n, double *partial, const int *done) {
  if (n <= 0) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_dot<T, KK>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, a, b, n, partial,
                                      done))
}

template <class T>
void launch_add_dot(hipStream_t stm, int K, const T *w, const T *r, T *z, int64_t row0, int64_t n, double *partial,
                    const int *done) {
  if (n <= 0) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_add_dot<T, KK>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, w, r, z, row0, n,
                                      partial, done))
}

template <class T>
void launch_jacobi(hipStream_t stm, int K, const T *r, const double *diag, T *z, int64_t n, const int *done) {
  if (n <= 0) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_jacobi<T, KK>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, r, diag, z, n,
                                      done))
}

void launch_gather(hipStream_t stm, int K, int k, const double *nat, const int64_t *perm, double *sto, int64_t n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_gather, grid(vec_blocks(n)), dim3(kBlock), 0, stm, nat, perm, sto, n, K, k);
}

void launch_scatter(hipStream_t stm, int K, int k, const double *sto, const int64_t *perm, double *nat, int64_t n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_scatter, grid(vec_blocks(n)), dim3(kBlock), 0, stm, sto, perm, nat, n, K, k);
}

void launch_gather_batch(hipStream_t stm, int K, const double *nat, int64_t N, const int64_t *perm, double *sto,
                         int64_t n, int cols) {
  if (n <= 0) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_gather_batch<KK>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, nat, N, perm,
                                      sto, n, cols))
}

void launch_scatter_batch(hipStream_t stm, int K, const double *sto, const int32_t *pos, double *nat, int64_t N,
                          int cols) {
  if (N <= 0) return;
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_scatter_batch<KK>), grid(vec_blocks(N)), dim3(kBlock), 0, stm, sto, pos, nat,
                                      N, cols))
}

void launch_demote(hipStream_t stm, int K, const double *r64, const double *scale, float *r32, int64_t n,
                   const int *done) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_demote, grid(vec_blocks(n * K)), dim3(kBlock), 0, stm, r64, scale, r32, n, K, done);
}

void launch_promote(hipStream_t stm, int K, const float *d32, const double *scale, double *x64, int64_t n,
                    const int *done) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_promote, grid(vec_blocks(n * K)), dim3(kBlock), 0, stm, d32, scale, x64, n, K, done);
}

void launch_pcg_init(hipStream_t stm, int K, Scal *s, const double *pb, int64_t npb, double tol, int maxit,
                     double *scale_in, double *scale_out) {
  hipLaunchKernelGGL(k_pcg_init, dim3(1), dim3(kBlock), 0, stm, s, pb, npb, K, tol, maxit, scale_in, scale_out);
}
void launch_pcg_set_rho(hipStream_t stm, int, Scal *s, const double *p, int64_t np) {
  hipLaunchKernelGGL(k_pcg_set_rho, dim3(1), dim3(kBlock), 0, stm, s, p, np);
}
// the per-iteration scalar kernels take K (= s->K) at compile time
void launch_compact(hipStream_t stm, int K, const double *p, int64_t np, double *out, const int *done) {
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_compact<KK>), dim3(kCompact), dim3(kBlock), 0, stm, p, np, out, done))
}
void launch_pcg_alpha(hipStream_t stm, int K, const Scal *in, Scal *mid, PartialSums pq) {
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_pcg_alpha<KK>), dim3(1), dim3(wide_block<KK>()), 0, stm, in, mid, pq.p,
                                      pq.n))
}
template <class T>
void launch_pcg_xr(hipStream_t stm, int K, const Scal *in, Scal *mid, PartialSums pq, T *x, T *r, const T *p,
                   const T *q, int64_t n, double *partial, float *r32, const double *scale) {
  auto run = [&](auto kernel, const Scal *s) {
    hipLaunchKernelGGL(kernel, grid(vec_blocks(n)), dim3(kBlock), 0, stm, s, mid, pq.p, pq.n, x, r, p, q, n, partial,
                       r32, scale);
  };
  VEMG_K_SWITCH(K, {
    if (pq.p)
      r32 ? run(k_pcg_xr<T, KK, true, true>, in) : run(k_pcg_xr<T, KK, true, false>, in);
    else
      r32 ? run(k_pcg_xr<T, KK, false, true>, mid) : run(k_pcg_xr<T, KK, false, false>, mid);
  })
}
void launch_pcg_conv(hipStream_t stm, int K, Scal *mid, PartialSums rr) {
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_pcg_conv<KK>), dim3(1), dim3(wide_block<KK>()), 0, stm, mid, rr.p, rr.n))
}
void launch_pcg_beta(hipStream_t stm, int K, const Scal *mid, Scal *in, PartialSums rz) {
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_pcg_beta<KK>), dim3(1), dim3(wide_block<KK>()), 0, stm, mid, in, rz.p,
                                      rz.n))
}
template <class T>
void launch_pcg_p(hipStream_t stm, int K, const Scal *mid, Scal *in, PartialSums rr, PartialSums rz, T *pvec,
                  const T *z, int64_t n) {
  auto run = [&](auto kernel, const Scal *s) {
    hipLaunchKernelGGL(kernel, grid(vec_blocks(n)), dim3(kBlock), 0, stm, s, in, rr.p, rr.n, rz.p, rz.n, pvec, z, n);
  };
  VEMG_K_SWITCH(K, {
    if (!rz.p)
      run(k_pcg_p<T, KK, false, false>, (const Scal *)in);
    else
      rr.p ? run(k_pcg_p<T, KK, true, true>, mid) : run(k_pcg_p<T, KK, true, false>, mid);
  })
}
void launch_promote_dot(hipStream_t stm, int K, const float *z32, const double *scale, const double *r, double *z64,
                        int64_t n, double *partial, const int *done) {
  VEMG_K_SWITCH(K, hipLaunchKernelGGL((k_promote_dot<KK>), grid(vec_blocks(n)), dim3(kBlock), 0, stm, z32, scale, r,
                                      z64, n, partial, done))
}
void launch_reduce(hipStream_t stm, int K, const double *p, int64_t np, double *out) {
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(kBlock), 0, stm, p, np, K, out);
}
void launch_pcg_resume(hipStream_t stm, int, Scal *s, unsigned keep) {
  hipLaunchKernelGGL(k_pcg_resume, dim3(1), dim3(64), 0, stm, s, keep);
}

#define VEMG_INSTANTIATE(T)                                                                                          \
  template void launch_spmv<T>(hipStream_t, int, const Sell &, int, int64_t, int64_t, const T *, T *, double *,       \
                               const int *, const SliceRef *);                                                       \
  template int64_t launch_gs<T>(hipStream_t, int, const Sell &, int64_t, int64_t, int64_t, int64_t, const T *, T *,    \
                                const int *, bool, double *);                                                        \
  template int64_t launch_gs_merged<T>(hipStream_t, int, const Sell &, const MergedRows &, int64_t, int64_t, int64_t,  \
                                       int64_t, int64_t, int64_t, const T *, T *, const int *, bool, double *);      \
  template void launch_res_merged<T>(hipStream_t, int, const Sell &, const MergedRows &, const T *, T *, const int *,  \
                                     const SliceRef *);                                                              \
  template void launch_prolong_merged<T>(hipStream_t, int, const MergedRows &, const T *, const T *, T *,             \
                                         const int *);                                                               \
  template void launch_rect<T>(hipStream_t, int, const Sell &, bool, const T *, T *, const int *);                    \
  template void launch_prolong_sum<T>(hipStream_t, int, const Sell &, int64_t, const T *, const T *, const T *, T *,   \
                                      double *, const int *);                                                        \
  template void launch_csr<T>(hipStream_t, int, CsrMode, const CsrJob<T> *, int, const int *);                            \
  template void launch_patch_gs<T>(hipStream_t, int, PatchDir, const PatchJob<T> *, int, const int *);                \
  template void launch_dense<T>(hipStream_t, int, const DenseJob<T> *, int, const int *);                             \
  template void launch_fill<T>(hipStream_t, T *, int64_t, T, const int *);                                           \
  template void launch_copy<T>(hipStream_t, const T *, T *, int64_t, const int *);                                   \
  template void launch_dot<T>(hipStream_t, int, const T *, const T *, int64_t, double *, const int *);                \
  template void launch_add_dot<T>(hipStream_t, int, const T *, const T *, T *, int64_t, int64_t, double *,             \
                                  const int *);                                                                      \
  template void launch_jacobi<T>(hipStream_t, int, const T *, const double *, T *, int64_t, const int *);             \
  template void launch_pcg_xr<T>(hipStream_t, int, const Scal *, Scal *, PartialSums, T *, T *, const T *, const T *,   \
                                 int64_t, double *, float *, const double *);                                        \
  template void launch_pcg_p<T>(hipStream_t, int, const Scal *, Scal *, PartialSums, PartialSums, T *, const T *,     \
                                int64_t);

VEMG_INSTANTIATE(double)
VEMG_INSTANTIATE(float)

}  // namespace vemg
