// Learned initial guess, reduced-basis part: a POD basis built by the
// method of snapshots from solutions the ensemble solver produced.
//
//   snapshots S [n][m] (one column per solved sample)
//   G = S^T S [m][m]                         (FP64 matrix cores, half of the symmetric product, split K)
//   top-r eigenpairs of G by block subspace iteration with a seeded start
//   block, orthonormalised between its steps (by a Cholesky factor, else by block
//   Gram-Schmidt), and a final Rayleigh-Ritz step after two rounds of block
//   Gram-Schmidt, whose k x k eigenproblem is solved by Jacobi rotations in
//   round-robin order in one workgroup
//   Phi = S V_r diag(lambda_r)^(-1/2) [n][r], each column's largest-magnitude
//   entry made positive
//   coefficients C = X^T Phi and reconstruction x0 = Phi c in the ensemble
//   layout [n][s].
// Everything is FP64 except the network outputs c (FP32).
#include "common.hpp"

namespace ens {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// C[M][N] = op(A)[M][K] B[K][N] in FP64 on the matrix cores
// (v_mfma_f64_16x16x4: lane l holds A[l%16][l/16] and B[l/16][l%16], the result
// leaves D[l/16 + 4 i][l%16], i = 0..3).  op(A)[i][k] is A[i*lda+k] (TA = 0) or
// A[k*lda+i] (TA = 1); B[k][j] is B[k*ldb+j].  A workgroup forms 128 x BN of C:
// BN = 128 as 2 x 2 wavefronts of 64 x 64, else four wavefronts of 32 x BN, so
// a step of 4 in k reads at most 8 operands from LDS for 16 MFMA (one a SIMD
// in 64 cycles) and the matrix cores, not LDS, bound the square products; the
// products with a narrow B (the basis and the projection, N = 32) are bound by
// reading A.  K slices of KS are staged k-major in LDS, double buffered, the
// next slice on its way in registers meanwhile.  blockIdx.z selects a K range
// [z*kchunk, (z+1)*kchunk) and writes its partial product to C + z*cstride.
// SYM (A = B): blockIdx.x counts the block pairs i <= j of the symmetric C,
// and with a single K range the mirrored block is written too.
// The Gram matrix of 2048 snapshots at 64^3: 18.4 ms (67 TFLOP/s of its
// half; a large library product reaches 72 here); with a bounds test around
// every load, workgroups in plain order and a last round of 12 in 512 it took
// 21.1 ms, the lane-per-4x4 form with all of C 70.9 ms.
template <int TA, int BN, int KS, bool SYM>
__global__ __launch_bounds__(256) void k_dgemm(int64_t M, int64_t N, int64_t K, const double* __restrict__ A,
                                               int64_t lda, const double* __restrict__ B, int64_t ldb,
                                               double* __restrict__ C, int64_t ldc, int64_t kchunk,
                                               int64_t cstride) {
  constexpr int BM = 128, WM = BN == 128 ? 64 : 32, WN = BN == 128 ? 64 : BN;
  constexpr int MT = WM / 16, NT = WN / 16, LA = BM + 2, LB = BN + 2;
  constexpr int UA = KS * BM / 256, UB = KS * BN / 256;
  __shared__ double As[2][KS * LA];
  __shared__ double Bs[2][KS * LB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, q = lane >> 4;
  const int wm = BN == 128 ? (wave >> 1) * 64 : wave * 32, wn = BN == 128 ? (wave & 1) * 64 : 0;
  int64_t bi = blockIdx.y, bj = blockIdx.x;
  uint32_t bz = blockIdx.z;
  if (SYM) {  // pair p -> (i, j), i <= j, column by column
    // workgroups are dealt to the 8 XCDs in turn: each XCD takes a run of the
    // pairs of one K range, whose rows of A then meet in its L2
    const uint32_t total = gridDim.x * gridDim.z, lin = bz * gridDim.x + blockIdx.x, xcd = lin % 8;
    const uint32_t at = xcd * (total / 8) + (xcd < total % 8 ? xcd : total % 8) + lin / 8;
    bz = at / gridDim.x;
    const int64_t p = at % gridDim.x;
    bj = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
    while (bj * (bj + 1) / 2 > p) --bj;
    while ((bj + 1) * (bj + 2) / 2 <= p) ++bj;
    bi = p - bj * (bj + 1) / 2;
  }
  const int64_t i0 = bi * BM, j0 = bj * BN;
  const int64_t kb = (int64_t)bz * kchunk;
  const int64_t ke = kb + kchunk < K ? kb + kchunk : K;
  double ra[UA], rb[UB];
  // rows and columns past the edge are read from the last one (what they give
  // is not stored), so only a K range's last slice needs a test per element
  const int ka = TA ? tid / BM : tid % KS, kbr = tid / BN;
  int64_t offa[TA ? 1 : UA];
#pragma unroll
  for (int u = 0; u < (TA ? 1 : UA); ++u) {
    const int64_t i = i0 + (TA ? tid % BM : (tid + 256 * u) / KS);
    offa[u] = TA ? ka * lda + (i < M ? i : M - 1) : (i < M ? i : M - 1) * lda + ka;
  }
  const int64_t jb = j0 + tid % BN, offb = kbr * ldb + (jb < N ? jb : N - 1);
  auto load = [&](int64_t k0) {
    const double* Ak = A + (TA ? k0 * lda : k0);
    const double* Bk = B + k0 * ldb;
    if (k0 + KS <= ke) {
#pragma unroll
      for (int u = 0; u < UA; ++u) ra[u] = TA ? (Ak + u * (256 / BM) * lda)[offa[0]] : Ak[offa[TA ? 0 : u]];
#pragma unroll
      for (int u = 0; u < UB; ++u) rb[u] = (Bk + u * (256 / BN) * ldb)[offb];
      return;
    }
    const int left = (int)(ke - k0);
#pragma unroll
    for (int u = 0; u < UA; ++u)
      ra[u] = ka + (TA ? u * (256 / BM) : 0) < left ? (TA ? (Ak + u * (256 / BM) * lda)[offa[0]] : Ak[offa[TA ? 0 : u]])
                                                    : 0.0;
#pragma unroll
    for (int u = 0; u < UB; ++u) rb[u] = kbr + u * (256 / BN) < left ? (Bk + u * (256 / BN) * ldb)[offb] : 0.0;
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const int t = tid + 256 * u;
      As[buf][(TA ? t / BM : t % KS) * LA + (TA ? t % BM : t / KS)] = ra[u];
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int t = tid + 256 * u;
      Bs[buf][(t / BN) * LB + t % BN] = rb[u];
    }
  };
  f64x4 acc[MT][NT];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[a][b] = (f64x4)0.0;
  load(kb);
  store(0);
  __syncthreads();
  int buf = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += KS, buf ^= 1) {
    const bool more = k0 + KS < ke;
    if (more) load(k0 + KS);
    // a wave that multiplies goes before one that loads, stores or leaves the
    // barrier: the two on a SIMD take turns (19.9 -> 18.3 ms)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < KS; kk += 4) {
      double a[MT], b[NT];
#pragma unroll
      for (int m = 0; m < MT; ++m) a[m] = As[buf][(kk + q) * LA + wm + 16 * m + r];
#pragma unroll
      for (int n = 0; n < NT; ++n) b[n] = Bs[buf][(kk + q) * LB + wn + 16 * n + r];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], b[n], acc[m][n], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  double* Cz = C + (int64_t)bz * cstride;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t i = i0 + wm + 16 * m + q + 4 * t, j = j0 + wn + 16 * n + r;
        if (i >= M || j >= N) continue;
        Cz[i * ldc + j] = acc[m][n][t];
        if (SYM && gridDim.z == 1 && bi != bj) Cz[j * ldc + i] = acc[m][n][t];
      }
}

// out[i] = sum_z parts[z*stride + i], z ascending.
__global__ void k_sum_slices(int64_t count, int nz, const double* __restrict__ parts, int64_t stride,
                             double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  double s = 0.0;
#pragma unroll 8
  for (int z = 0; z < nz; ++z) s += parts[(int64_t)z * stride + i];
  out[i] = s;
}

// The same for a symmetric m x m product whose slices hold the blocks i <= j of
// 128 x 128 only: a workgroup sums a 32 x 32 piece of one and writes it and
// its mirror image, turned over in LDS.
__global__ __launch_bounds__(256) void k_sum_slices_sym(int64_t m, int nz, const double* __restrict__ parts,
                                                        int64_t stride, double* __restrict__ out) {
  const int64_t i0 = (int64_t)blockIdx.y * 32, j0 = (int64_t)blockIdx.x * 32;
  if (i0 / 128 > j0 / 128) return;
  __shared__ double t[32][33];
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = i0 + g + 8 * u, j = j0 + c;
    if (i < m && j < m) {
      double s = 0.0;
#pragma unroll 8
      for (int z = 0; z < nz; ++z) s += parts[(int64_t)z * stride + i * m + j];
      out[i * m + j] = s;
      t[g + 8 * u][c] = s;
    }
  }
  if (i0 / 128 == j0 / 128) return;  // a diagonal block holds both halves
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t j = j0 + g + 8 * u, i = i0 + c;
    if (i < m && j < m) out[j * m + i] = t[c][g + 8 * u];
  }
}

// Orthonormalise the k columns of Y [m][k] (row-major) in place: block
// Gram-Schmidt over panels of 16 columns, each panel taken twice through
// "project out the panels before it, then orthonormalise it inside", which
// leaves the columns orthonormal to rounding (the second round finds them so
// to about 1e-11 and cleans up).  Between two power steps a basis that close
// to orthonormal does as well, so there (`once`) the second round is left out
// for a panel whose columns kept at least 1 % of their length in the first.  One
// workgroup of 8 wavefronts does it all: the time is a chain of reductions over m, and Y (1 MB for 2048 x 64) stays
// in L2.  Projections, panel Gram matrices and the updates are 16 x 16 tiles
// on the FP64 matrix cores, whose reads of Y are whole 128-byte pieces of
// rows; the columns one at a time, each product a strided pass, took 11.1 ms
// for 2048 x 64, now 0.58 ms, and 0.30 ms with one round a panel.
// Inside a panel: Y R^-1 from the Cholesky factor of its Gram matrix (columns
// scaled to length one first) when every column keeps at least 1 % of its
// length off the columns before it, so the factor is accurate; otherwise
// column by column, classical Gram-Schmidt twice each, which also takes
// columns that are dependent to rounding (a zero column stays zero).
constexpr int kPanel = 16;
constexpr int kOrthWaves = 8, kOrthThreads = 64 * kOrthWaves;
constexpr double kCholeskyMin = 1e-4;  // least squared length off the columns before

struct OrthLds {
  double red[kOrthWaves][256];            // per-wavefront tiles or sums
  double d[256 * kPanel];         // projections onto the columns before the panel
  double w[kPanel * kPanel];      // the panel's Gram matrix
  double rinv[kPanel * kPanel];
  double col[kPanel];
  int ok, clean;  // Cholesky is accurate; and the projection left every column most of its length
};

// Tiles t0 .. t0 + NT - 1 of X^T Yp, X the columns 16 t of Y (PANEL: Yp
// itself), into out[16 (t - t0) + i][j].
template <int NT, bool PANEL>
__device__ inline void orth_dots(int m, int k, const double* Y, int t0, int j0, int b, OrthLds& s, double* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  f64x4 acc[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) acc[u] = (f64x4)0.0;
  for (int row0 = 4 * wave; row0 < m; row0 += 16 * kOrthWaves) {  // the operands of four steps in flight
    double bv[4], av[4][NT];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = row0 + 4 * kOrthWaves * v + q;
      const double* yr = Y + (int64_t)row * k;
      bv[v] = (row < m && r < b) ? yr[j0 + r] : 0.0;
#pragma unroll
      for (int u = 0; u < NT; ++u) av[v][u] = PANEL ? bv[v] : (row < m ? yr[16 * (t0 + u) + r] : 0.0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int u = 0; u < NT; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[v][u], bv[v], acc[u], 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < NT; ++u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s.red[wave][(q + 4 * i) * 16 + r] = acc[u][i];
    __syncthreads();
    if (threadIdx.x < 256) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < kOrthWaves; ++w) v += s.red[w][threadIdx.x];
      out[u * 256 + threadIdx.x] = v;
    }
    __syncthreads();
  }
}

// R^-1 of the panel's Gram matrix by elimination on [W | 1] in the registers
// of one wavefront: lane (row i = lane % 16, columns 8 (lane / 16) .. + 7).
// Sets s.ok and s.clean (j0 columns were projected out).
__device__ inline void orth_cholesky(int j0, int b, OrthLds& s) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  // unit columns; columns past the panel count as unit vectors of their own
  const double wii = i < b ? s.w[i * 17] : 1.0;
  const double sc = 1.0 / sqrt(wii);
  double a[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const int c = 8 * g + v;
    const double sj = __shfl(sc, c & 15, 64);
    a[v] = c >= 16 ? (c - 16 == i ? 1.0 : 0.0)
                   : (i == c ? 1.0 : (i < b && c < b ? s.w[i * 16 + c] * sc * sj : 0.0));
  }
  bool ok = wii > 0.0 && wii < INFINITY;
  double dii = 1.0;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const double piv = __shfl(a[p & 7], p + 16 * (p >> 3), 64);
    const double f = __shfl(a[p & 7], i + 16 * (p >> 3), 64) / piv;
    ok = ok && piv >= kCholeskyMin;
    if (i == p) dii = piv;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const double pr = __shfl(a[v], p + 16 * g, 64);
      if (i > p) a[v] -= f * pr;
    }
  }
  const double rs = 1.0 / sqrt(dii);
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const int l = (8 * g + v) & 15;
    const double sl = __shfl(sc, l, 64);
    if (g >= 2) s.rinv[l * 16 + i] = a[v] * rs * sl;
  }
  double off = 0.0;  // what the projection took off column i, squared
  for (int row = g; row < j0; row += 4) off += s.d[row * 16 + i] * s.d[row * 16 + i];
  off += __shfl_xor(off, 16, 64);
  off += __shfl_xor(off, 32, 64);
  const int all_ok = __all(ok), all_clean = __all(ok && wii >= kCholeskyMin * off);
  if (lane == 0) {
    s.ok = all_ok;
    s.clean = all_clean;
  }
}

// Block-wide sums of v[0 .. n-1] over the workgroup's lanes, to s.col.
template <int NV>
__device__ inline void orth_sums(const double (&v)[NV], int n, OrthLds& s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (i < n) {
      double t = v[i];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
      if (lane == 0) s.red[wave][i] = t;
    }
  __syncthreads();
  if ((int)threadIdx.x < n) {
    double t = 0.0;
    for (int w = 0; w < kOrthWaves; ++w) t += s.red[w][threadIdx.x];
    s.col[threadIdx.x] = t;
  }
  __syncthreads();
}

// done (nullable): nonzero when the columns are orthonormal already.
__global__ __launch_bounds__(kOrthThreads) void k_orth(int m, int k, double* Y, int once, const int* done) {
  if (done && *done) return;
  __shared__ OrthLds s;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, r = lane & 15, q = lane >> 4;
  const int tiles = (m + 15) / 16;
  for (int j0 = 0; j0 < k; j0 += kPanel) {
    const int b = k - j0 < kPanel ? k - j0 : kPanel;
    for (int round = 0; round < 2; ++round) {
      if (j0 > 0) {
        int t0 = 0;
        for (; t0 + 2 <= j0 / 16; t0 += 2) orth_dots<2, false>(m, k, Y, t0, j0, b, s, s.d + t0 * 256);
        for (; t0 < j0 / 16; ++t0) orth_dots<1, false>(m, k, Y, t0, j0, b, s, s.d + t0 * 256);
        for (int tl = wave; tl < tiles; tl += kOrthWaves) {
          const int ra = 16 * tl + r;
          f64x4 acc;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = 16 * tl + q + 4 * i;
            acc[i] = (row < m && r < b) ? Y[(int64_t)row * k + j0 + r] : 0.0;
          }
          for (int k0 = 0; k0 < j0; k0 += 16) {
            double av[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) av[v] = ra < m ? -Y[(int64_t)ra * k + k0 + 4 * v + q] : 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v)
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[v], s.d[(k0 + 4 * v + q) * 16 + r], acc, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = 16 * tl + q + 4 * i;
            if (row < m && r < b) Y[(int64_t)row * k + j0 + r] = acc[i];
          }
        }
        __syncthreads();
      }
      orth_dots<1, true>(m, k, Y, 0, j0, b, s, s.w);
      if (wave == 0) orth_cholesky(j0, b, s);
      __syncthreads();
      if (s.ok) {
        for (int tl = wave; tl < tiles; tl += kOrthWaves) {
          const int ra = 16 * tl + r;
          f64x4 acc = (f64x4)0.0;
#pragma unroll
          for (int kk = 0; kk < 16; kk += 4) {
            const double av = (ra < m && kk + q < b) ? Y[(int64_t)ra * k + j0 + kk + q] : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, s.rinv[(kk + q) * 16 + r], acc, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = 16 * tl + q + 4 * i;
            if (row < m && r < b) Y[(int64_t)row * k + j0 + r] = acc[i];
          }
        }
      } else {
        for (int j = 0; j < b; ++j) {
          for (int pass = 0; pass < 2 && j > 0; ++pass) {
            double acc[kPanel];
#pragma unroll
            for (int i = 0; i < kPanel; ++i) acc[i] = 0.0;
#pragma unroll 1
            for (int row = t; row < m; row += kOrthThreads) {
              const double* yr = Y + (int64_t)row * k + j0;
              const double yj = yr[j];
#pragma unroll
              for (int i = 0; i < kPanel; ++i)
                if (i < j) acc[i] += yr[i] * yj;
            }
            orth_sums(acc, j, s);
            for (int row = t; row < m; row += kOrthThreads) {
              double* yr = Y + (int64_t)row * k + j0;
              double v = yr[j];
              for (int i = 0; i < j; ++i) v -= s.col[i] * yr[i];
              yr[j] = v;
            }
          }
          double sq[1] = {0.0};
          for (int row = t; row < m; row += kOrthThreads) {
            const double v = Y[(int64_t)row * k + j0 + j];
            sq[0] += v * v;
          }
          orth_sums(sq, 1, s);
          const double nrm = sqrt(s.col[0]), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
          for (int row = t; row < m; row += kOrthThreads) Y[(int64_t)row * k + j0 + j] *= inv;
          __syncthreads();
        }
      }
      const int done = once && s.clean;
      __syncthreads();
      if (done) break;
    }
  }
}

// Jacobi on a symmetric k x k matrix H (row-major, in place), one workgroup;
// on exit the diagonal of H holds the eigenvalues and U [k][k] the
// eigenvectors (columns).  A sweep is k - 1 rounds (k even; an odd one has an
// idle index) of k / 2 rotations of disjoint pairs, the round-robin order: the
// angles of a round come from one lane each, then every 2 x 2 block of rows
// of one pair and columns of another is rotated from both sides by one lane,
// so a round is two barriers where the cyclic order takes three for each of
// its rotations.  Sweeps end when one rotates nothing (entries at most 1e-18
// of their diagonals' geometric mean), at most `sweeps`.  H and U lie in LDS
// up to k = 96 (LDS: 2 k^2 doubles).  k = 64: 0.48 ms, against 11.6 ms for the
// cyclic order's 12 sweeps in L2.
constexpr int kJacobiLdsK = 96;

// U = R^-1 for the Cholesky factor R of H = Y^T Y [k][k], k <= kJacobiLdsK, so
// that Y U is orthonormal: all columns of a power step at once, where each keeps
// at least 1 % of its length off the columns before it (as they do once the
// first steps have sorted the eigenvectors; Q then is orthonormal to about
// 1e-11, which serves between power steps).  Otherwise U = I and *done = 0, and
// k_orth takes over.  One workgroup: the elimination [A | I] -> [R | L^-1] of the
// matrix scaled to a unit diagonal, in LDS, k steps of one rank-one update, bound
// by their chain (42 us for k = 64).  With the products Y^T Y and Y U over all of
// the chip, orth(Y) of 2048 x 64 so takes 75 us, against 390 us in k_orth, whose one
// workgroup passes over all rows; of 12 power steps the first needs k_orth.
__global__ __launch_bounds__(1024) void k_cholesky_inverse(int k, const double* __restrict__ H,
                                                           double* __restrict__ U, int* __restrict__ done) {
  constexpr int kG = 16;  // wavefronts
  extern __shared__ double s_chol[];
  double* A = s_chol;                // [k][k + 1]
  double* W = s_chol + k * (k + 1);  // [k][k + 1]
  __shared__ double s_d[kJacobiLdsK];
  const int t = threadIdx.x, ld = k + 1;
  if (t < k) {
    const double h = H[(int64_t)t * k + t];
    s_d[t] = h > 0.0 ? 1.0 / sqrt(h) : 0.0;
  }
  __syncthreads();
  for (int x = t; x < k * k; x += 64 * kG) {
    const int i = x / k, j = x % k;
    A[i * ld + j] = H[x] * s_d[i] * s_d[j];
    W[i * ld + j] = i == j ? 1.0 : 0.0;
  }
  __syncthreads();
  const int c = t & 63, g = t >> 6;  // columns c and c + 64 of every kG-th row
  bool ok = true;
  for (int j = 0; j < k; ++j) {
    const double p = A[j * ld + j];
    ok = p >= 1e-4;  // (false for NaN)
    if (!ok) break;
    const double inv = 1.0 / p;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x = c + 64 * h;
      if (x >= k) break;
      // columns past j of A, up to j of W (its rows are L's inverse, unscaled)
      double* const M = (x > j ? A : W) + x;
      const double top = -inv * M[j * ld];
      for (int i0 = j + 1 + g; i0 < k; i0 += 4 * kG) {  // four rows in flight
        double f[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = i0 + u * kG < k ? i0 + u * kG : k - 1;
          f[u] = A[i * ld + j];
          v[u] = M[i * ld];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i0 + u * kG < k) M[(i0 + u * kG) * ld] = fma(f[u], top, v[u]);
      }
    }
    __syncthreads();
  }
  if (t == 0) *done = ok;
  for (int x = t; x < k * k; x += 64 * kG) {
    const int i = x / k, j = x % k;  // U[i][j] = W[j][i] / sqrt(pivot j) in the scaled columns
    U[x] = !ok ? (i == j ? 1.0 : 0.0) : i <= j ? s_d[i] * W[j * ld + i] / sqrt(A[j * ld + j]) : 0.0;
  }
}

template <bool LDS>
__global__ __launch_bounds__(1024) void k_jacobi(int k, double* Hg, double* Ug, int sweeps) {
  extern __shared__ double s_hu[];
  __shared__ double s_c[128], s_s[128];
  __shared__ short s_p[128], s_q[128];
  __shared__ int s_any;
  double* H = LDS ? s_hu : Hg;
  double* U = LDS ? s_hu + k * k : Ug;
  const int t = threadIdx.x, nt = blockDim.x;
  const int k2 = k + (k & 1), pairs = k2 / 2;
  for (int i = t; i < k * k; i += nt) {
    if (LDS) H[i] = Hg[i];
    U[i] = (i / k == i % k) ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int sw = 0; sw < sweeps; ++sw) {
    if (t == 0) s_any = 0;
    for (int round = 0; round < k2 - 1; ++round) {
      __syncthreads();
      if (t < pairs) {
        // round-robin: index k2 - 1 stays, the others move round by one
        const int x = t == 0 ? k2 - 1 : (round + t) % (k2 - 1);
        const int y = (round + (k2 - 1) - t) % (k2 - 1);
        const int p = x < y ? x : y, q = x < y ? y : x;
        double c = 1.0, s = 0.0;
        if (q < k) {
          const double apq = H[p * k + q], app = H[p * k + p], aqq = H[q * k + q];
          if (!(fabs(apq) <= 1e-300 || fabs(apq) <= 1e-18 * sqrt(fabs(app * aqq)))) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + tt * tt);
            s = tt * c;
            s_any = 1;
          }
        }
        s_p[t] = (short)p;
        s_q[t] = (short)q;
        s_c[t] = c;
        s_s[t] = s;
      }
      __syncthreads();
      for (int i = t; i < pairs * pairs; i += nt) {
        const int a = i / pairs, b = i % pairs;
        const double ca = s_c[a], sa = s_s[a], cb = s_c[b], sb = s_s[b];
        if (sa == 0.0 && sb == 0.0) continue;
        const int p = s_p[a], q = s_q[a], u = s_p[b], v = s_q[b];
        const bool qk = q < k, vk = v < k;
        // rows p, q by the pair a's rotation, then columns u, v by b's
        const double hpu = H[p * k + u], hpv = vk ? H[p * k + v] : 0.0;
        const double hqu = qk ? H[q * k + u] : 0.0, hqv = qk && vk ? H[q * k + v] : 0.0;
        const double rpu = ca * hpu - sa * hqu, rpv = ca * hpv - sa * hqv;
        const double rqu = sa * hpu + ca * hqu, rqv = sa * hpv + ca * hqv;
        const bool own = a == b;  // its off-diagonal entries are what the rotation removes
        H[p * k + u] = cb * rpu - sb * rpv;
        if (vk) H[p * k + v] = own && sa != 0.0 ? 0.0 : sb * rpu + cb * rpv;
        if (qk) H[q * k + u] = own && sa != 0.0 ? 0.0 : cb * rqu - sb * rqv;
        if (qk && vk) H[q * k + v] = sb * rqu + cb * rqv;
      }
      for (int i = t; i < k * pairs; i += nt) {
        const int row = i / pairs, b = i % pairs;
        const double cb = s_c[b], sb = s_s[b];
        if (sb == 0.0) continue;
        const int u = s_p[b], v = s_q[b];
        const double up = U[row * k + u], uq = U[row * k + v];
        U[row * k + u] = cb * up - sb * uq;
        U[row * k + v] = sb * up + cb * uq;
      }
    }
    __syncthreads();
    const int any = s_any;
    __syncthreads();
    if (!any) break;
  }
  if (LDS)
    for (int i = t; i < k * k; i += nt) {
      Hg[i] = H[i];
      Ug[i] = U[i];
    }
}

// Sort the Jacobi result by eigenvalue descending (equal ones by index);
// V[m][r] = Q U[:, top r], lambda[r].
__global__ __launch_bounds__(256) void k_ritz_select(int m, int k, int r, const double* __restrict__ H,
                                                     const double* __restrict__ U, const double* __restrict__ Q,
                                                     double* __restrict__ V, double* __restrict__ lambda) {
  __shared__ double diag[256];
  __shared__ int order[256];
  const int t = threadIdx.x;  // k <= 256
  order[t] = 0;               // (a NaN ranks nowhere)
  if (t < k) diag[t] = H[t * k + t];
  __syncthreads();
  if (t < k) {
    int rank = 0;
    for (int j = 0; j < k; ++j) rank += diag[j] > diag[t] || (diag[j] == diag[t] && j < t);
    order[rank] = t;
  }
  __syncthreads();
  if (blockIdx.x == 0 && t < r) lambda[t] = diag[order[t]];
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + t; x < (int64_t)m * r; x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = x / r;
    const int c = order[x % r];
    double s = 0.0;
    for (int l = 0; l < k; ++l) s += Q[i * k + l] * U[l * k + c];
    V[x] = s;
  }
}

// Phi columns scaled by lambda^(-1/2), in place on the S V product, with the
// sign rule: the largest-magnitude entry of every column is positive (ties: the
// lowest row).  One workgroup per column; each of its loads touches as many
// lines as it has lanes, and the rate at which one CU takes such misses bounds
// it (1.05 ms at 64^3 for reading twice and writing once; 1.18 ms for the sign
// alone with one load in flight a lane, and a pass of its own for the scale).
__global__ __launch_bounds__(1024) void k_scale_sign_cols(int64_t n, int r, double* __restrict__ P,
                                                          const double* __restrict__ lambda) {
  constexpr int NT = 1024, D = 8;
  __shared__ double bv[NT / 64], bs[NT / 64];
  __shared__ int64_t bi[NT / 64];
  const int j = blockIdx.x, t = threadIdx.x;
  const double inv = 1.0 / sqrt(lambda[j]);
  double best = -1.0, bval = 0.0;
  int64_t besti = 0;
  for (int64_t i0 = t; i0 < n; i0 += NT * D) {
    double v[D];
#pragma unroll
    for (int d = 0; d < D; ++d) v[d] = i0 + NT * d < n ? P[(i0 + NT * d) * r + j] : 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const double a = v[d] * inv;
      if (i0 + NT * d < n && fabs(a) > best) {
        best = fabs(a);
        bval = a;
        besti = i0 + NT * d;
      }
    }
  }
  auto take = [&](double o, double ov, int64_t oi) {
    if (o > best || (o == best && oi < besti)) {
      best = o;
      bval = ov;
      besti = oi;
    }
  };
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(best, off, 64), ov = __shfl_xor(bval, off, 64);
    const int64_t oi = __shfl_xor((long long)besti, off, 64);
    take(o, ov, oi);
  }
  if ((t & 63) == 0) {
    bv[t >> 6] = best;
    bs[t >> 6] = bval;
    bi[t >> 6] = besti;
  }
  __syncthreads();
  best = bv[0];
  bval = bs[0];
  besti = bi[0];
  for (int w = 1; w < NT / 64; ++w) take(bv[w], bs[w], bi[w]);
  const bool flip = bval < 0.0;
  for (int64_t i0 = t; i0 < n; i0 += NT * D) {
    double v[D];
#pragma unroll
    for (int d = 0; d < D; ++d) v[d] = i0 + NT * d < n ? P[(i0 + NT * d) * r + j] : 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (i0 + NT * d < n) P[(i0 + NT * d) * r + j] = flip ? -(v[d] * inv) : v[d] * inv;
  }
}

// S[i][col0 + e] = x[i][e]
__global__ void k_collect(int64_t n, int s, const double* __restrict__ x, double* __restrict__ S, int m, int col0) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * s) return;
  const int64_t i = t / s;
  const int e = (int)(t % s);
  S[i * m + col0 + e] = x[t];
}

// x0[i][e] = sum_j Phi[i][j] (mu[j] + sd[j] c[e][j])   (c FP32; mu, sd nullable)
__device__ inline double destandardised(const float* __restrict__ c, const double* __restrict__ mu,
                                        const double* __restrict__ sd, int64_t at, int j) {
  double cj = (double)c[at];
  if (sd) cj *= sd[j];
  if (mu) cj += mu[j];
  return cj;
}

// One lane per entry, the coefficients of all samples staged once per block,
// sample fastest: the lanes of a wavefront read neighbouring samples (kept
// by sample, each lane's stride of r doubles put all of them on one bank).
__global__ __launch_bounds__(256) void k_reconstruct(int64_t n, int r, int s, const double* __restrict__ Phi,
                                                     const float* __restrict__ c, const double* __restrict__ mu,
                                                     const double* __restrict__ sd, double* __restrict__ x0) {
  extern __shared__ double chat[];
  for (int t = threadIdx.x; t < s * r; t += blockDim.x) {
    const int j = t % r;
    chat[j * s + t / r] = destandardised(c, mu, sd, t, j);
  }
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * s) return;
  const int64_t i = t / s;
  const int e = (int)(t % s);
  const double* prow = Phi + i * r;
  double acc = 0.0;
  for (int j = 0; j < r; ++j) acc += prow[j] * chat[j * s + e];
  x0[t] = acc;
}

// The same product on the FP64 matrix cores (v_mfma_f64_16x16x4): a wavefront
// forms 16 nodes x 32 samples at a time.  It is bound by reading Phi and
// writing x0, so the layout is the loads': the four k values of an MFMA step
// are free to choose, and with k = 32 c + 8 (lane / 16) + t a lane's operands
// are 8 consecutive entries of one row of Phi (four 16-byte loads, every
// 64-byte piece of the row used whole).  The coefficients lie in LDS in the
// order the lanes take them.  Measured at 64^3, r = s = 32, where Phi and x0
// (141 MB) fit the last-level cache: 26 us from there (5.4 TB/s), 32 us where the
// buffers change from call to call and come from memory (4.4 TB/s), against 475 us
// both ways for the lane-per-entry form with its bank conflicts.
// MFMA layout: lane l holds A[l%16][l/16] and B[l/16][l%16]; the result
// leaves D[l/16 + 4 i][l%16], i = 0..3.
constexpr int kRecMaxR = 256;  // 64 KB of coefficients in LDS

__global__ __launch_bounds__(256) void k_reconstruct_mfma(int64_t n, int r, int s, const double* __restrict__ Phi,
                                                          const float* __restrict__ c, const double* __restrict__ mu,
                                                          const double* __restrict__ sd, double* __restrict__ x0) {
  extern __shared__ double frag[];  // [tile of 16 samples][chunk][t][lane]
  const int chunks = (r + 31) / 32, e0 = blockIdx.y * 32;
  for (int t = threadIdx.x; t < 2 * chunks * 512; t += blockDim.x) {
    const int l = t & 63, step = (t >> 6) & 7, ck = (t >> 9) % chunks, tile = t / (chunks * 512);
    const int e = e0 + 16 * tile + (l & 15), j = 32 * ck + 8 * (l >> 4) + step;
    frag[t] = (e < s && j < r) ? destandardised(c, mu, sd, (int64_t)e * r + j, j) : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, q = lane >> 4, col = lane & 15;
  const int64_t tiles = (n + 15) / 16;
  for (int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); w < tiles; w += (int64_t)gridDim.x * 4) {
    const int64_t row = w * 16 + col;
    f64x4 acc[2] = {(f64x4)0.0, (f64x4)0.0};
    for (int ck = 0; ck < chunks; ++ck) {
      const int j0 = 32 * ck + 8 * q;
      f64x2 a[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        a[v] = (row < n && j0 < r) ? *(const f64x2*)(Phi + row * r + j0 + 2 * v) : (f64x2)0.0;
      const double* f = frag + ck * 512 + lane;
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int g = 0; g < 2; ++g)
          acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t >> 1][t & 1], f[(g * chunks * 8 + t) * 64], acc[g], 0, 0, 0);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t node = w * 16 + q + 4 * i;
        const int e = e0 + 16 * g + col;
        if (node < n && e < s) x0[node * s + e] = acc[g][i];
      }
  }
}

// Mean and standard deviation of each coefficient over the m snapshots, the
// scale of each coefficient its own deviation or (common) the largest of them,
// and the network targets T = (C - mu) / scale.  With one common scale the
// targets keep the coefficients' relative sizes, so the network's squared
// error is the squared error of the lifted guess in the orthonormal basis.
// One workgroup: 1024 / r lanes a coefficient, each on a stride of the rows,
// their sums added in lane order (one lane a coefficient: 980 us for 2048 x 32,
// now 33 us).
__global__ __launch_bounds__(1024) void k_standardize(int m, int r, int common, const double* __restrict__ C,
                                                      double* __restrict__ mu, double* __restrict__ sd,
                                                      float* __restrict__ T) {
  __shared__ double s_part[1024];
  __shared__ double s_mean[1024], s_dev[1024];
  const int t = threadIdx.x, G = 1024 / r, j = t % r, g = t / r;
  const bool live = g < G;
  auto column_sum = [&](auto term) -> double {  // the column's sum, for the lanes t < r
    double s = 0.0;
    if (live) {
      int i = g;
      for (; i + 3 * G < m; i += 4 * G) {
        const double v0 = C[(int64_t)i * r + j], v1 = C[(int64_t)(i + G) * r + j];
        const double v2 = C[(int64_t)(i + 2 * G) * r + j], v3 = C[(int64_t)(i + 3 * G) * r + j];
        s += (term(v0) + term(v1)) + (term(v2) + term(v3));
      }
      for (; i < m; i += G) s += term(C[(int64_t)i * r + j]);
    }
    s_part[t] = s;
    __syncthreads();
    double tot = 0.0;
    if (t < r)
      for (int h = 0; h < G; ++h) tot += s_part[h * r + t];
    __syncthreads();
    return tot;
  };
  const double s1 = column_sum([](double v) { return v; });
  if (t < r) s_mean[t] = s1 / m;
  __syncthreads();
  const double mean = s_mean[j];
  const double s2 = column_sum([&](double v) { return (v - mean) * (v - mean); });
  if (t < r) s_dev[t] = sqrt(s2 / m);
  __syncthreads();
  double dev = s_dev[j];
  if (common) {
    double mx = 0.0;
    for (int i = 0; i < r; ++i) mx = s_dev[i] > mx ? s_dev[i] : mx;
    dev = mx;
  }
  if (!(dev > 0.0)) dev = 1.0;
  if (t < r) {
    mu[t] = mean;
    sd[t] = dev;
  }
  if (live)
    for (int i = g; i < m; i += G) T[(int64_t)i * r + j] = (float)((C[(int64_t)i * r + j] - mean) / dev);
}

// ------------------------------------------------------------ host side ---

// K ranges a product of `tiles` workgroup tiles is split into: as many as make
// `want` workgroups (about 512 are resident), none under 128 of K (a sum pass
// reads each range's product again), at most 128.
static int k_splits(int64_t tiles, int64_t K, int64_t want) {
  int64_t s = (want + tiles - 1) / tiles, most = K / 128;
  if (most > 128) most = 128;
  if (s > most) s = most;
  return (int)(s < 1 ? 1 : s);
}

static int64_t tiles128(int64_t n) { return (n + 127) / 128; }

// The widest tile of the three that N fills.
static int tile_n(int64_t N) { return N <= 32 ? 32 : N <= 64 ? 64 : 128; }

static int product_splits(int64_t M, int64_t N, int64_t K) {
  const int bn = tile_n(N);
  return k_splits(tiles128(M) * ((N + bn - 1) / bn), K, 1024);
}

// Ranges of the Gram product: of the counts that give 2 to 8 rounds of the 512
// workgroups the chip holds at once the one whose last round is fullest, the
// fewest ranges of equals (2048 snapshots at 64^3: 31 ranges leave the last round
// almost empty, 21.1 ms; 30 and 15 fill it, 20.4 ms).
static int gram_splits(int64_t n, int64_t m) {
  const int64_t t = tiles128(m), pairs = t * (t + 1) / 2;
  const int most = k_splits(pairs, n, 4096);
  int best = most;
  double fill = 0.0;
  for (int s = most; 4 * s >= most; --s) {
    const int64_t rounds = (pairs * s + 511) / 512;
    const double f = (double)(pairs * s) / (double)(rounds * 512);
    if (f >= fill) {
      fill = f;
      best = s;
    }
  }
  return best;
}

// Ranges that a product over n rows takes with the workspace it is given, `slice`
// bytes a range: `want` where it holds them, fewer where it does not.  Refused
// is a workspace of fewer than n / 4096 ranges (32 at most, `want` at most); none
// is needed where that is one.
static ens_status ranges_held(int want, int64_t n, size_t slice, const void* ws, size_t ws_bytes, int* ranges) {
  int64_t least = n / 4096 < 32 ? n / 4096 : 32;
  if (least > want) least = want;
  ENS_ARG_CHECK(least <= 1 || ws, "null workspace");
  const int64_t held = ws ? (int64_t)(ws_bytes / slice) : 0;
  if (least > 1 && held < least) {
    set_error("workspace of %zu bytes is smaller than the %zu required", ws_bytes, (size_t)least * slice);
    return ENS_E_NOMEM;
  }
  *ranges = held < 1 ? 1 : held < want ? (int)held : want;
  return ENS_OK;
}

// C [M][N] (dense) = op(A) B in `splits` K ranges; scratch [splits][M][N] for
// more than one.
template <int TA>
static void dgemm(int64_t M, int64_t N, int64_t K, const double* A, int64_t lda, const double* B, int64_t ldb,
                  double* C, int splits, double* scratch, hipStream_t st) {
  int64_t kchunk = (K + splits - 1) / splits;
  kchunk = (kchunk + 31) / 32 * 32;
  const int nz = (int)((K + kchunk - 1) / kchunk);
  double* out = nz > 1 ? scratch : C;
  const int bn = tile_n(N);
  const dim3 grid((unsigned)((N + bn - 1) / bn), (unsigned)tiles128(M), (unsigned)nz);
  if (bn == 32)
    hipLaunchKernelGGL((k_dgemm<TA, 32, 16, false>), grid, dim3(256), 0, st, M, N, K, A, lda, B, ldb, out, N, kchunk,
                       M * N);
  else if (bn == 64)
    hipLaunchKernelGGL((k_dgemm<TA, 64, 16, false>), grid, dim3(256), 0, st, M, N, K, A, lda, B, ldb, out, N, kchunk,
                       M * N);
  else
    hipLaunchKernelGGL((k_dgemm<TA, 128, 16, false>), grid, dim3(256), 0, st, M, N, K, A, lda, B, ldb, out, N, kchunk,
                       M * N);
  if (nz > 1)
    hipLaunchKernelGGL(k_sum_slices, dim3((unsigned)((M * N + 255) / 256)), dim3(256), 0, st, M * N, nz, scratch,
                       M * N, C);
}

// Doubles of workspace the eigensolver cannot do without, and those of its
// products' split-K scratch.
static size_t eig_least(int64_t m, int64_t k) { return 3 * (size_t)m * k + 3 * (size_t)k * k + 64; }
static size_t eig_scratch(int64_t m, int64_t k) {
  const size_t a = (size_t)product_splits(m, k, m) * m * k, b = (size_t)product_splits(k, k, m) * k * k;
  return a > b ? a : b;
}

}  // namespace ens

using namespace ens;

extern "C" {

ens_status ens_pod_collect(const double* x, int64_t n, int32_t s, double* S, int32_t m, int32_t col0,
                           hipStream_t stream) {
  ENS_ARG_CHECK(x && S && n >= 0 && s >= 1 && m >= 1 && col0 >= 0 && col0 + s <= m, "bad collect arguments");
  if (n == 0) return ENS_OK;
  hipLaunchKernelGGL(k_collect, dim3((unsigned)((n * s + 255) / 256)), dim3(256), 0, stream, n, s, x, S, m, col0);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_gram_workspace_bytes(int64_t n, int32_t m, size_t* bytes) {
  ENS_ARG_CHECK(bytes && n >= 1 && m >= 1, "bad sizes");
  *bytes = (size_t)gram_splits(n, m) * m * m * sizeof(double);
  return ENS_OK;
}

ens_status ens_pod_gram(const double* S, int64_t n, int32_t m, double* G, void* workspace, size_t ws_bytes,
                        hipStream_t stream) {
  ENS_ARG_CHECK(S && G && n >= 1 && m >= 1, "bad Gram arguments");
  int sp = 1;
  const ens_status rc = ranges_held(gram_splits(n, m), n, (size_t)m * m * sizeof(double), workspace, ws_bytes, &sp);
  if (rc != ENS_OK) return rc;
  // G = S^T S: op(A) = S^T, K = n; the blocks on and above the diagonal
  const int64_t tm = tiles128(m), m64 = m;
  const int64_t kchunk = ((n + sp - 1) / sp + 31) / 32 * 32;
  const int nz = (int)((n + kchunk - 1) / kchunk);
  double* parts = (double*)workspace;
  hipLaunchKernelGGL((k_dgemm<1, 128, 16, true>), dim3((unsigned)(tm * (tm + 1) / 2), 1, (unsigned)nz), dim3(256), 0,
                     stream, m64, m64, n, S, m64, S, m64, nz > 1 ? parts : G, m64, kchunk, m64 * m64);
  if (nz > 1)
    hipLaunchKernelGGL(k_sum_slices_sym, dim3((unsigned)((m + 31) / 32), (unsigned)((m + 31) / 32)), dim3(256), 0,
                       stream, m64, nz, parts, m64 * m64, G);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_eig_workspace_bytes(int32_t m, int32_t k, size_t* bytes) {
  ENS_ARG_CHECK(bytes && m >= 1 && k >= 1, "bad sizes");
  *bytes = (eig_least(m, k) + eig_scratch(m, k)) * sizeof(double);
  return ENS_OK;
}

ens_status ens_pod_eig(const double* G, int32_t m, int32_t k, int32_t r, const double* start, int32_t iters,
                       double* V, double* lambda, void* workspace, size_t ws_bytes, hipStream_t stream) {
  ENS_ARG_CHECK(G && start && V && lambda && workspace, "null pointer");
  ENS_ARG_CHECK(m >= 1 && k >= 1 && k <= 256 && k <= m && r >= 1 && r <= k && iters >= 0, "bad sizes");
  const size_t least = eig_least(m, k);
  if (ws_bytes < least * sizeof(double)) {
    set_error("eigen workspace too small");
    return ENS_E_NOMEM;
  }
  double* Y = (double*)workspace;
  double* Q = Y + (size_t)m * k;
  double* T = Q + (size_t)m * k;
  double* H = T + (size_t)m * k;
  double* U = H + (size_t)k * k;
  double* parts = U + 2 * (size_t)k * k + 64;
  // K ranges as far as the workspace holds their products
  const size_t room = ws_bytes / sizeof(double) - least;
  auto held = [&](int want, size_t product) {
    return room < product ? 1 : room / product < (size_t)want ? (int)(room / product) : want;
  };
  const int sy = held(product_splits(m, k, m), (size_t)m * k), sh = held(product_splits(k, k, m), (size_t)k * k);
  ENS_HIP_TRY(hipMemcpyAsync(Y, start, (size_t)m * k * sizeof(double), hipMemcpyDeviceToDevice, stream));
  // power steps: Y <- G orth(Y); orth(Y) from the factor of Y^T Y where it serves
  int* const done = (int*)(U + 2 * (size_t)k * k);
  for (int it = 0; it < iters; ++it) {
    if (k <= kJacobiLdsK) {
      dgemm<1>(k, k, m, Y, k, Y, k, H, sh, parts, stream);
      hipLaunchKernelGGL(k_cholesky_inverse, dim3(1), dim3(1024), 2 * (size_t)k * (k + 1) * sizeof(double), stream, k,
                         H, U, done);
      dgemm<0>(m, k, k, Y, k, U, k, Q, 1, nullptr, stream);
      hipLaunchKernelGGL(k_orth, dim3(1), dim3(kOrthThreads), 0, stream, m, k, Q, 1, done);
      dgemm<0>(m, k, m, G, m, Q, k, Y, sy, parts, stream);
      continue;
    }
    hipLaunchKernelGGL(k_orth, dim3(1), dim3(kOrthThreads), 0, stream, m, k, Y, 1, (const int*)nullptr);
    dgemm<0>(m, k, m, G, m, Y, k, Q, sy, parts, stream);
    double* const tmp = Y;
    Y = Q;
    Q = tmp;
  }
  // Rayleigh-Ritz on span(Y)
  hipLaunchKernelGGL(k_orth, dim3(1), dim3(kOrthThreads), 0, stream, m, k, Y, 0, (const int*)nullptr);
  dgemm<0>(m, k, m, G, m, Y, k, T, sy, parts, stream);   // T = G Q
  dgemm<1>(k, k, m, Y, k, T, k, H, sh, parts, stream);   // H = Q^T G Q
  if (k <= kJacobiLdsK)
    hipLaunchKernelGGL(k_jacobi<true>, dim3(1), dim3(1024), 2 * (size_t)k * k * sizeof(double), stream, k, H, U, 12);
  else
    hipLaunchKernelGGL(k_jacobi<false>, dim3(1), dim3(1024), 0, stream, k, H, U, 12);
  hipLaunchKernelGGL(k_ritz_select, dim3(64), dim3(256), 0, stream, m, k, r, H, U, Y, V, lambda);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_basis(const double* S, int64_t n, int32_t m, const double* V, const double* lambda, int32_t r,
                         double* Phi, hipStream_t stream) {
  ENS_ARG_CHECK(S && V && lambda && Phi && n >= 1 && m >= 1 && r >= 1 && r <= m, "bad basis arguments");
  dgemm<0>(n, r, m, S, m, V, r, Phi, 1, nullptr, stream);  // Phi = S V
  hipLaunchKernelGGL(k_scale_sign_cols, dim3((unsigned)r), dim3(1024), 0, stream, n, r, Phi, lambda);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_project_workspace_bytes(int64_t n, int32_t r, int32_t s, size_t* bytes) {
  ENS_ARG_CHECK(bytes && n >= 1 && r >= 1 && s >= 1, "bad sizes");
  *bytes = (size_t)product_splits(s, r, n) * r * s * sizeof(double);
  return ENS_OK;
}

ens_status ens_pod_project(const double* Phi, const double* X, int64_t n, int32_t r, int32_t s, double* C,
                           void* workspace, size_t ws_bytes, hipStream_t stream) {
  ENS_ARG_CHECK(Phi && X && C && n >= 1 && r >= 1 && s >= 1, "bad projection arguments");
  int sp = 1;
  const ens_status rc = ranges_held(product_splits(s, r, n), n, (size_t)r * s * sizeof(double), workspace, ws_bytes, &sp);
  if (rc != ENS_OK) return rc;
  // C[e][j] = sum_i X[i][e] Phi[i][j]: op(A) = X^T
  dgemm<1>(s, r, n, X, s, Phi, r, C, sp, (double*)workspace, stream);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_reconstruct(const double* Phi, int64_t n, int32_t r, const float* c, const double* mu,
                               const double* sd, int32_t s, double* x0, hipStream_t stream) {
  ENS_ARG_CHECK(Phi && c && x0 && n >= 1 && r >= 1 && s >= 1, "bad reconstruction arguments");
  ENS_ARG_CHECK((int64_t)s * r <= 8192, "s * r must not exceed 8192 (coefficients staged in 64 KB of LDS)");
  // The matrix-core form takes rows of Phi as 16-byte loads of whole
  // 8-entry groups (r a multiple of 8, Phi 16-byte aligned), r up to its LDS,
  // and at least 8 of a tile's 16 samples live; the rest go one lane an entry.
  if (r % 8 == 0 && r <= kRecMaxR && s >= 8 && aligned16(Phi)) {
    const int64_t blocks = (n + 63) / 64;
    hipLaunchKernelGGL(k_reconstruct_mfma, dim3((unsigned)(blocks < 1024 ? blocks : 1024), (unsigned)((s + 31) / 32)),
                       dim3(256), (size_t)(r + 31) / 32 * 1024 * sizeof(double), stream, n, r, s, Phi, c, mu, sd, x0);
  } else {
    hipLaunchKernelGGL(k_reconstruct, dim3((unsigned)((n * s + 255) / 256)), dim3(256),
                       (size_t)s * r * sizeof(double), stream, n, r, s, Phi, c, mu, sd, x0);
  }
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_pod_standardize(const double* C, int32_t m, int32_t r, int32_t common, double* mu, double* sd,
                               float* T, hipStream_t stream) {
  ENS_ARG_CHECK(C && mu && sd && T && m >= 1 && r >= 1 && r <= 1024, "bad standardize arguments");
  hipLaunchKernelGGL(k_standardize, dim3(1), dim3(1024), 0, stream, m, r, common, C, mu, sd, T);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

}  // extern "C"
