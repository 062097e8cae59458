// Device building blocks of the ensemble sparse products (Sec. 2).
//
// Fig. "ensemble_crs" puts the sample loop innermost: for each stored entry
// the column index is read once and the s-long ensembles of the value and of
// x[col] are contiguous.  On a 64-wide wavefront we map that inner loop onto
// lanes: one 16-byte load holds V = 16/sizeof(T) samples, L = s/V lanes
// cover one entry's ensemble, and KS such lane groups share a row, taking
// every KS-th entry; the groups' sums are added by a butterfly.  With one
// group a row, a narrow ensemble is read in pieces of L * 16 bytes a row and
// the 27 entries are nine dependent rounds of three loads; KS groups read KS
// entries of a row side by side in as many fewer rounds, at the price of the
// butterfly and of vector work on only 1/KS of the lanes (row_groups below
// says when it pays).  The values stream is read with non-temporal loads so
// it does not evict the reused x entries from the caches.
#pragma once

#include "common.hpp"

namespace ens {

// Lane groups per row.  Ensembles of 64 bytes or less (L <= 4) always gain
// from several groups; wider ones gain with 4 while the matrix fits the 256 MB
// last-level cache (SMALL: latency counts), and beyond that, where HBM bounds
// the pass, a little with 2, or not at all where the pass also forms sums of
// its rows for a reduction (DOT: the shorter tiles write more partials).
// Measured, one group -> this many (us):
//   product        64^3: FP64 s = 4 107 -> 54, 8 123 -> 90, 16 165 -> 158, 32 327
//                  -> 318; FP32 s = 4 110 -> 35, 8 106 -> 54, 16 120 -> 90;
//                  128^3: FP32 s = 32 1375 -> 1354
//   smoother pass  8^3, 16^3, 32^3: FP32 s = 32 7.9 -> 4.4, 8.3 -> 5.7, 29.0 ->
//                  24.6; FP64 s = 16 the same; 64^3: FP64 s = 16 184 -> 177, s = 8
//                  130 -> 100; 128^3: FP32 s = 32 1510 -> 1475
//   with DOT       32^3: FP64 s = 16 28.6 -> 25.8; 64^3: s = 8 131 -> 105; s = 16
//                  186 with one, 183 to 188 with 2 and 4; 128^3: FP32 s = 32 1526
//                  with one, 1554 with 2
// (FP32 sums take at most 4: the workspace of a refinement holds 2 S partials
// for every 512 / S rows.)
template <typename T, int S, bool DOT, bool SMALL>
constexpr int row_groups() {
  constexpr int L = S * (int)sizeof(T) / 16;
  if (L <= 4) return L == 4 || (DOT && sizeof(T) == 4) ? 4 : 8;
  return SMALL ? 4 : DOT ? 1 : 2;
}

// Whether an ensemble matrix of nnz entries fits the last-level cache.
template <typename T, int S>
inline bool cached_matrix(int64_t nnz) {
  return nnz * (int64_t)(S * sizeof(T)) <= ((int64_t)256 << 20);
}

template <typename T, int S, int KSv = 1>
struct EnsMap {
  static constexpr int V = pack<T>::V;  // samples per 16-byte load
  static_assert(S % V == 0, "ensemble size must fill a 16-byte load");
  static constexpr int L = S / V;       // lanes per entry
  static constexpr int KS = KSv;        // lane groups per row
  static constexpr int W = L * KS;      // lanes per row
  static constexpr int RPW = 64 / W;    // rows per wavefront
  typedef typename pack<T>::type vt;
};

template <typename VT>
__device__ inline VT load_stream(const VT* p) {
  return __builtin_nontemporal_load(p);
}

// Streamed results are written with non-temporal stores: in a
// read-dominated stream the ordinary write-back stores cost far more read
// bandwidth than their few bytes (measured about 3.5 % of SpMV throughput).
template <typename VT>
__device__ inline void store_stream(VT* p, VT v) {
  __builtin_nontemporal_store(v, p);
}

// A workgroup's row tile staged in LDS: the row offsets of rows r0..r0+R
// and the column indices of their entries, read once per workgroup with
// coalesced loads (one index per lane instead of one per L-lane group and
// entry), after which the lanes take their indices from LDS.  Measured at
// 128^3, s = 32 in FP32: the CG product 5.08 -> 5.36 TB/s and the multigrid
// row passes 5.23 -> 5.46 TB/s against the per-lane index loads.  CAP = 32
// indices per row covers the 27-point rows with room; a tile whose entries
// do not fit (other graphs) reads its indices from global memory.
template <int R>
constexpr int kTileCap = R * 32;

template <int R, int CAP = kTileCap<R>>
struct RowTileLds {
  int32_t rp[R + 1];
  int32_t ci[CAP];
};

// Stage rows r0 .. min(r0 + R, n) - 1 (every lane of the workgroup calls
// this).  Returns false, staging only the offsets, when their entries do not
// fit in CAP indices; the caller then reads the indices from global memory.
template <int R, int CAP>
__device__ inline bool stage_row_tile(RowTileLds<R, CAP>& t, int n, const int32_t* __restrict__ rp,
                                      const int32_t* __restrict__ ci, int64_t r0) {
  const int rows = (int)((int64_t)n - r0 < R ? (int64_t)n - r0 : R);
  for (int i = threadIdx.x; i <= rows; i += blockDim.x) t.rp[i] = rp[r0 + i];
  __syncthreads();
  const int64_t base = t.rp[0], cnt = (int64_t)t.rp[rows] - base;
  if (cnt > CAP) return false;
  for (int i = threadIdx.x; i < (int)cnt; i += blockDim.x) t.ci[i] = ci[base + i];
  __syncthreads();
  return true;
}

// sum_k vals[k] x[ci[k]] over the entries k0 .. k1 of a row for the V samples
// of lane `sub`, in precision TA (TV and TX widened as they are read): lane
// group g of KS takes the entries k0 + g, k0 + g + KS, ..., and the butterfly
// over the groups leaves the sum in every one.  The loads of a split row are
// predicated one by one, U in flight; with the row unrolled whole and every
// load issued at once the same products ran 6 to 10 % slower.
template <int S, int V, int KS, typename TA, typename TV, typename TX>
__device__ inline typename vec_t<TA, V>::type row_sum(const int32_t* ci, const TV* __restrict__ vals,
                                                      const TX* __restrict__ x, int64_t k0, int64_t k1, int sub,
                                                      int g) {
  constexpr int L = S / V;
  typedef typename vec_t<TV, V>::type av;
  typedef typename vec_t<TX, V>::type xv;
  typename vec_t<TA, V>::type acc = (typename vec_t<TA, V>::type)0;
  const av* vv = (const av*)vals + sub;
  const xv* xx = (const xv*)x + sub;
  if constexpr (KS == 1) {
    int64_t k = k0;
    for (; k + 2 < k1; k += 3) {
      int32_t c[3];
      av a[3];
      xv b[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) c[j] = ci[k + j];
#pragma unroll
      for (int j = 0; j < 3; ++j) a[j] = load_stream(vv + (k + j) * L);
#pragma unroll
      for (int j = 0; j < 3; ++j) b[j] = xx[(int64_t)c[j] * L];
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += (TA)a[j][v] * (TA)b[j][v];
    }
    for (; k < k1; ++k) {
      const av a = load_stream(vv + k * L);
      const xv b = xx[(int64_t)ci[k] * L];
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += (TA)a[v] * (TA)b[v];
    }
  } else {
    constexpr int U = KS == 2 ? 9 : 4;
    for (int64_t k = k0 + g; k < k1; k += KS * U) {
      av a[U];
      xv b[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u * KS < k1) a[u] = load_stream(vv + (k + u * KS) * L);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u * KS < k1) b[u] = xx[(int64_t)ci[k + u * KS] * L];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u * KS < k1)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[v] += (TA)a[u][v] * (TA)b[u][v];
    }
#pragma unroll
    for (int off = L; off < L * KS; off <<= 1)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += __shfl_xor(acc[v], off, 64);
  }
  return acc;
}

// Row tile of a workgroup.  Workgroups are dealt to the 8 XCDs in turn; runs of
// 16 consecutive tiles go to one XCD where the gathered vector is 16 MB or less
// (n rows of S samples in T), so that neighbouring rows read it through one L2
// (product, us: 27^3, FP64 s = 8 9.2 -> 8.9, 32^3, FP32 s = 16 14.3 -> 13.6, 48^3,
// FP64 s = 16 73.3 -> 70.8).  A larger vector does not stay in the L2s, and the
// matrix then streams best in launch order (96^3, FP32 s = 32 544 -> 553 in runs,
// 128^3 1342 -> 1364).
template <typename T, int S>
__device__ inline int64_t row_tile(int n) {
  constexpr uint32_t C = 16;
  const uint32_t b = blockIdx.x, run = b / (8 * C), in = b % (8 * C);
  if ((int64_t)n * (S * (int)sizeof(T)) > ((int64_t)16 << 20) || (run + 1) * (8 * C) > gridDim.x) return b;
  return run * (8 * C) + (in % 8) * C + in / 8;
}

// A lane's place in a row tile of NW wavefronts: its samples sub*V .., lane
// group g (the one with g = 0 does the row's vector work) and row.
template <typename T, int S, int KS, int NW>
struct RowPlace {
  using M = EnsMap<T, S, KS>;
  static constexpr int R = NW * M::RPW;  // rows per tile
  int sub, g, lr;
  __device__ inline RowPlace() {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    sub = lane % M::L;
    g = (lane / M::L) % KS;
    lr = wave * M::RPW + lane / M::W;
  }
};

// Row product of a lane's row of the tile through the staged indices when
// they were staged, else from global memory.  (t.ci - t.rp[0])[k] is entry k's
// index.
template <typename TA, typename T, int S, int KS, int NW, typename TV, typename TX, int R, int CAP>
__device__ inline typename vec_t<TA, EnsMap<T, S>::V>::type tile_row_product(const RowPlace<T, S, KS, NW>& at,
                                                                             const RowTileLds<R, CAP>& t, bool staged,
                                                                             const int32_t* __restrict__ ci,
                                                                             const TV* __restrict__ vals,
                                                                             const TX* __restrict__ x) {
  constexpr int V = EnsMap<T, S>::V;
  const int64_t k0 = t.rp[at.lr], k1 = t.rp[at.lr + 1];
  if (staged) return row_sum<S, V, KS, TA>(t.ci - t.rp[0], vals, x, k0, k1, at.sub, at.g);
  return row_sum<S, V, KS, TA>(ci, vals, x, k0, k1, at.sub, at.g);
}

// Block-wide per-sample reduction of NQ quantities over NW wavefronts.
// Each lane holds vals[q][j] for samples sub*VS + j (j < VS); lanes with
// equal (lane % L) hold the same samples.  The block totals are written to
// dst[q][s] (one row of the partial array) in a fixed order.
template <int S, int VS, int NQ, int NW>
__device__ inline void block_partials(double (&vals)[NQ][VS], double* __restrict__ dst) {
  constexpr int L = S / VS;
  __shared__ double red[NW][NQ][S];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int j = 0; j < VS; ++j) {
      double v = wave_sum_stride<L>(vals[q][j]);
      if (lane < L) red[wave][q][lane * VS + j] = v;
    }
  __syncthreads();
  if (threadIdx.x < NQ * S) {
    const int q = threadIdx.x / S, e = threadIdx.x % S;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w][q][e];
    dst[q * S + e] = t;
  }
}

// dst[qe] = sum over r < rows of src[r*P + qe] for the P columns of a
// row-major partial array: the rows are split into G = 256/P interleaved
// stripes, which are added by a butterfly within each wavefront and in wavefront
// order afterwards.  The order depends only on `rows`, so the result is
// bit-reproducible.  Bound by its chain: eight loads in flight a lane, and no
// serial pass over the stripes (64 of them at P = 4: the update of a 16^3, s = 4
// solve, which sums 308 rows before it starts, 7.3 -> 6.4 us).
template <int P>
__device__ inline void sum_rows(const double* __restrict__ src, int64_t rows, double* __restrict__ dst) {
  static_assert(P <= 64 && 64 % P == 0, "whole stripes in a wavefront");
  constexpr int G = kBlock / P, NW = kBlock / 64;
  __shared__ double wsum[NW][P];
  const int t = threadIdx.x;
  const int g = t / P, qe = t % P;
  constexpr int D = 8;
  double a[D];
#pragma unroll
  for (int d = 0; d < D; ++d) a[d] = 0.0;
  for (int64_t r = g; r < rows; r += D * G) {
    double v[D];
#pragma unroll
    for (int d = 0; d < D; ++d) v[d] = r + d * G < rows ? src[(r + d * G) * P + qe] : 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) a[d] += v[d];
  }
  const double v = wave_sum_stride<P>(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
  if ((t & 63) < P) wsum[t >> 6][qe] = v;
  __syncthreads();
  if (t < P) {
    double acc = wsum[0][t];
#pragma unroll
    for (int w = 1; w < NW; ++w) acc += wsum[w][t];
    dst[t] = acc;
  }
  __syncthreads();
}

}  // namespace ens
