// Ensemble Q1 assembly of the stiffness matrix and load vector.
//
// Alg. "assembly" (Sec. 4) loops over cells and scatters each element matrix
// into the global matrix with atomic adds.  Here the loop is turned inside
// out: a lane owns one matrix row (one node) of one sample, visits the 8
// elements around an interior node in ascending element id and adds the
// element row K_e[a_i][.] into a 27-entry register row (a boundary row is an
// identity row and needs none).  No atomics are needed, each entry sums its
// elements in ascending order, and since every K_e is formed from a symmetric
// table with the same operations for (a,b) and (b,a) the assembled matrix is
// bitwise symmetric.
// The coefficient at each element's Gauss points is evaluated once per
// workgroup tile into LDS (k_assemble_tile).  The writes of a row are
// sample-contiguous ([nnz][s]).
//
// Element matrix on the uniform mesh (h = 1/N, 2x2x2 Gauss, weight h^3/8):
//   K_e[a][b] = sum_q kappa_q (h/8) G_q[a][b],
//   G_q[a][b] = grad_ref N_a(g_q) . grad_ref N_b(g_q)       (dimensionless)
// kappa_q = kappa0 + sigma sum_m sqrt(lambda_m) phi_m(x_q) y_m, with the 1D
// factors of phi_m read from the KL table.
#include "common.hpp"
#include "mg.hpp"

namespace ens {

constexpr int kAsmMaxM = 16;

// Q1 element tables at the 2 x 2 x 2 Gauss points (Sec. 4, Alg. assembly),
// fixed at compile time: with the element loops unrolled every entry the
// kernels read is a known constant, and since the reference coordinate of
// a Gauss point along each axis is (1 -+ 1/sqrt 3)/2 the tables hold only
// a few distinct values, which the compiler keeps in registers instead of
// loading (and spilling) a table per element.
struct Q1Tables {
  double G[8][8][8];   // [q][a][b]: grad N_a . grad N_b (reference), symmetric in (a,b)
  double dN[8][8][3];  // [q][a][d]: reference derivative of N_a along axis d
};

constexpr Q1Tables q1_tables() {
  Q1Tables t{};
  const double r = 0.57735026918962576451;
  const double g[2] = {0.5 * (1.0 - r), 0.5 * (1.0 + r)};
  for (int q = 0; q < 8; ++q) {
    const double s3[3] = {g[q & 1], g[(q >> 1) & 1], g[(q >> 2) & 1]};
    for (int a = 0; a < 8; ++a) {
      const int ax[3] = {a & 1, (a >> 1) & 1, (a >> 2) & 1};
      double l[3] = {0.0, 0.0, 0.0}, d[3] = {0.0, 0.0, 0.0};
      for (int k = 0; k < 3; ++k) {
        l[k] = ax[k] ? s3[k] : 1.0 - s3[k];
        d[k] = ax[k] ? 1.0 : -1.0;
      }
      t.dN[q][a][0] = d[0] * l[1] * l[2];
      t.dN[q][a][1] = l[0] * d[1] * l[2];
      t.dN[q][a][2] = l[0] * l[1] * d[2];
    }
    for (int a = 0; a < 8; ++a)
      for (int b = a; b < 8; ++b) {
        double dot = 0.0;
        for (int k = 0; k < 3; ++k) dot += t.dN[q][a][k] * t.dN[q][b][k];
        t.G[q][a][b] = dot;
        t.G[q][b][a] = dot;
      }
  }
  return t;
}

__device__ constexpr Q1Tables kQ1 = q1_tables();

// Node tiles of the assemblies: a workgroup owns R = TX x TY x TZ nodes
// (one lane per row and sample); the elements touching the tile form an
// EX x EY x EZ block.
template <int Rv, int TYv>
struct AsmTile {
  static constexpr int R = Rv;
  static constexpr int TY = TYv, TZ = 4, TX = R / (TY * TZ);
  static constexpr int EX = TX + 1, EY = TY + 1, EZ = TZ + 1, NE = EX * EY * EZ;
  static_assert(TX * TY * TZ == R, "tile shape");
};

// LDS slot of Gauss point q of tile element le (of NE) for sample sb: point by
// point, so that the lanes of a wavefront, which read the same q of consecutive
// elements, hit different banks and all points lie at fixed offsets of one.
template <int NE, int SB>
__device__ inline int kslot(int le, int q, int sb) {
  return (q * NE + le) * SB + sb;
}

// LDS doubles of a tile's KL factors: the 1D eigenfunctions of the M modes at
// the 2 Gauss abscissae of each element column along x (by their x index), y
// and z (by mode).
template <int EX, int EY, int EZ>
__host__ __device__ constexpr int tab_doubles(int M) { return M * 2 * (EX + EY + EZ); }

// Phase 1 of the tiled assemblies: the coefficient at the 8 Gauss points of
// every element of the tile's EX x EY x EZ element block (origin ex0, ey0,
// ez0) for the SB samples e0.., times `scale`, into s_k[kslot(le, q, sb)].
// The 1D factors are staged in s_tab first, and each lane keeps the
// coefficients c_m = scale sigma sqrt(lambda_m) y_m of its one sample in registers
// (the NT lanes are a multiple of SB, so a lane's items all have the same
// sample).  An item is one sample's half column of elements along x: the modes
// with the same x factor X_i collapse into one weight for each of the column's
// 4 (y, z) Gauss lines,
//   W_i = sum over the modes m with x index i of c_m Y_m Z_m,
// scale kappa = scale kappa0 + sum_i X_i W_i, kColSlots x indices at a time (the 10 leading
// modes have 3).  Half columns of 3 and 2 elements: 30 items a sample for the 32
// lanes; with an element an item every mode cost its multiply-adds at every
// point, 120 operations instead of about 37 an element at 10 modes, and three
// times the LDS reads.  Ends with a barrier.
constexpr int kColSlots = 3;

template <int NT, int SB, int EX, int EY, int EZ>
__device__ __forceinline__ void tile_coefficients(int N, const double* __restrict__ kl_sqrt_lam,
                                         const int32_t* __restrict__ kl_triple, const double* __restrict__ kl_phi,
                                         int M, double kappa0, double sigma, const double* __restrict__ xi, int e0,
                                         int ex0, int ey0, int ez0, double scale, double* s_tab, double* s_k) {
  constexpr int HX = (EX + 1) / 2;  // elements of a half column (the second may hold one less)
  static_assert(NT % SB == 0 && 2 * EY * EZ <= NT / SB, "an item a lane, all of a lane's of one sample");
  const int64_t two_n = 2 * (int64_t)N;
  double* s_x = s_tab;             // [x index][EX][2]
  double* s_y = s_x + M * 2 * EX;  // [M][EY][2]
  double* s_z = s_y + M * 2 * EY;  // [M][EZ][2]
  for (int t = threadIdx.x; t < M * 2 * (EX + EY + EZ); t += NT) {
    int64_t k, at;
    if (t < M * 2 * EX) {
      k = t / (2 * EX);
      at = 2 * (int64_t)ex0 + t % (2 * EX);
    } else if (t < M * 2 * (EX + EY)) {
      const int r = t - M * 2 * EX;
      k = kl_triple[3 * (r / (2 * EY)) + 1];
      at = 2 * (int64_t)ey0 + r % (2 * EY);
    } else {
      const int r = t - M * 2 * (EX + EY);
      k = kl_triple[3 * (r / (2 * EZ)) + 2];
      at = 2 * (int64_t)ez0 + r % (2 * EZ);
    }
    s_tab[t] = at >= 0 && at < two_n ? kl_phi[k * two_n + at] : 0.0;
  }
  const int sb = threadIdx.x % SB;
  double c[kAsmMaxM];
#pragma unroll
  for (int m = 0; m < kAsmMaxM; ++m) c[m] = m < M ? scale * sigma * kl_sqrt_lam[m] * xi[(int64_t)(e0 + sb) * M + m] : 0.0;
  int nx = 0;  // x indices in use: 0 .. nx - 1
  for (int m = 0; m < M; ++m) nx = kl_triple[3 * m] >= nx ? kl_triple[3 * m] + 1 : nx;
  __syncthreads();
  const int col = (threadIdx.x / SB) >> 1, lx0 = (threadIdx.x / SB) & 1 ? HX : 0;
  const int ly = col % EY, lz = col / EY;
  const int ey = ey0 + ly, ez = ez0 + lz;
  if (lz < EZ && ey >= 0 && ez >= 0 && ey < N && ez < N) {
    double kq[HX][8];  // Gauss points qx + 2 (qy + 2 qz)
#pragma unroll
    for (int l = 0; l < HX; ++l)
#pragma unroll
      for (int q = 0; q < 8; ++q) kq[l][q] = kappa0 * scale;
    for (int i0 = 0; i0 < nx; i0 += kColSlots) {
      double w[kColSlots][4];
#pragma unroll
      for (int i = 0; i < kColSlots; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[i][j] = 0.0;
      // every mode up to the largest M, each skipped by a uniform branch
      // when absent: the coefficients stay in fixed registers
#pragma unroll
      for (int m = 0; m < kAsmMaxM; ++m) {
        if (m < M) {
          const int slot = kl_triple[3 * m] - i0;
          const double* py = s_y + (m * EY + ly) * 2;
          const double* pz = s_z + (m * EZ + lz) * 2;
          const double y0 = py[0], y1 = py[1], z0 = c[m] * pz[0], z1 = c[m] * pz[1];
#pragma unroll
          for (int i = 0; i < kColSlots; ++i)
            if (slot == i) {
              w[i][0] = fma(y0, z0, w[i][0]);
              w[i][1] = fma(y1, z0, w[i][1]);
              w[i][2] = fma(y0, z1, w[i][2]);
              w[i][3] = fma(y1, z1, w[i][3]);
            }
        }
      }
#pragma unroll
      for (int i = 0; i < kColSlots; ++i) {
        if (i0 + i < nx) {
#pragma unroll
          for (int l = 0; l < HX; ++l) {
            // (the slot past a shorter half's last element is read, not used)
            const double* px = s_x + ((i0 + i) * EX + lx0 + l) * 2;
            const double f0 = px[0], f1 = px[1];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              kq[l][2 * j] = fma(f0, w[i][j], kq[l][2 * j]);
              kq[l][2 * j + 1] = fma(f1, w[i][j], kq[l][2 * j + 1]);
            }
          }
        }
      }
    }
#pragma unroll
    for (int l = 0; l < HX; ++l) {
      const int lx = lx0 + l, ex = ex0 + lx;
      if (lx < EX && ex >= 0 && ex < N) {
        const int le = lx + EX * (ly + EY * lz);
#pragma unroll
        for (int q = 0; q < 8; ++q) s_k[kslot<EX * EY * EZ, SB>(le, q, sb)] = kq[l][q];
      }
    }
  }
  __syncthreads();
}

// Workgroup index -> (tile, sample group, tile origin).  Workgroups are
// dealt to the 8 XCDs round-robin by index; the G sample groups of one tile
// take indices 8 apart (same XCD, dispatched together) so their partial
// writes of each row's sample ensemble meet in one L2.
template <int TX, int TY, int TZ, int G>
__device__ inline void tile_decode(int N, uint32_t bid, int64_t* tile_id, int* sg, int* x0, int* y0, int* z0) {
  const uint32_t n1 = N + 1;
  const uint32_t ntx = (n1 + TX - 1) / TX, nty = (n1 + TY - 1) / TY, ntz = (n1 + TZ - 1) / TZ;
  const uint32_t tiles = ntx * ntz * nty;  // fits: at most 257 x 513 x 257
  uint32_t tile;
  if (G > 1 && (bid / (8 * G)) < tiles / 8) {
    const uint32_t blk = bid / (8 * G), rem = bid % (8 * G);
    *sg = (int)(rem / 8);
    tile = blk * 8 + rem % 8;
  } else {
    const uint32_t rest = bid - (tiles / 8) * 8 * G;  // the last tiles % 8 tiles, plainly
    *sg = (int)(G > 1 ? rest % G : 0);
    tile = (G > 1 ? (tiles / 8) * 8 + rest / G : bid);
  }
  *tile_id = tile;
  *x0 = (int)(tile % ntx) * TX;
  tile /= ntx;
  *z0 = (int)(tile % ntz) * TZ;
  *y0 = (int)(tile / ntz) * TY;
}

// Advection of one node's row, scale times sum_q N_a (v.dN_b) / 8 over its eight
// elements, for the 27 neighbours into s_adv: products over the axes of what
// the two elements of an axis add up to, the 1D mass (1/6, 2/3, 1/6) and first
// derivative (-1/2, 0, 1/2); the same for every interior row.
__device__ inline void advection_entries(double scale, double vx, double vy, double vz, double* s_adv) {
  if (threadIdx.x >= 27) return;
  const int d[3] = {(int)threadIdx.x % 3, ((int)threadIdx.x / 3) % 3, (int)threadIdx.x / 9};
  double m[3], g[3];
  for (int k = 0; k < 3; ++k) {
    m[k] = d[k] == 1 ? 2.0 / 3.0 : 1.0 / 6.0;
    g[k] = 0.5 * (d[k] - 1);
  }
  s_adv[threadIdx.x] = scale * (vx * (g[0] * m[1] * m[2]) + vy * (m[0] * g[1] * m[2]) + vz * (m[0] * m[1] * g[2]));
}

// Off-diagonal diffusion entries of an interior row (rx, ry, rz of the tile,
// sample sbl) from its four elements below (EZO -1) or above (0) the node,
// added to acc[neighbour] in ascending element order.  l_0 l_1 is the same at
// both Gauss points of an axis, so grad N_a . grad N_b does not depend on the
// point's position along the axes in which a and b differ: the coefficient is
// summed along those first (38 operations an element instead of 56).
template <typename T, int SB, int EZO>
__device__ __forceinline__ void diffusion_elements(const double* s_k, int rx, int ry, int rz, int sbl,
                                                   double (&acc)[27]) {
  const double* sk = s_k + kslot<T::NE, SB>(rx + T::EX * (ry + T::EY * (rz + 1 + EZO)), 0, sbl);
#pragma unroll
  for (int ey_off = -1; ey_off <= 0; ++ey_off)
#pragma unroll
    for (int ex_off = -1; ex_off <= 0; ++ex_off) {
      const int ai = (-ex_off) + 2 * (-ey_off) + 4 * (-EZO);
      double kq[8], sx[4], sy[4], sz[4];
#pragma unroll
      for (int q = 0; q < 8; ++q) kq[q] = sk[kslot<T::NE, SB>(1 + ex_off + T::EX * (1 + ey_off), q, 0)];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sx[j] = kq[2 * j] + kq[2 * j + 1];                              // j = qy + 2 qz
        sy[j] = kq[(j & 1) + 4 * (j >> 1)] + kq[(j & 1) + 4 * (j >> 1) + 2];  // qx + 2 qz
        sz[j] = kq[j] + kq[j + 4];                                      // qx + 2 qy
      }
      const double sxy[2] = {sx[0] + sx[1], sx[2] + sx[3]};  // by qz
      const double sxz[2] = {sx[0] + sx[2], sx[1] + sx[3]};  // by qy
      const double syz[2] = {sy[0] + sy[2], sy[1] + sy[3]};  // by qx
      auto entry = [&](int b) -> double& {
        return acc[(EZO + (b >> 2) + 1) * 9 + (ey_off + ((b >> 1) & 1) + 1) * 3 + ex_off + (b & 1) + 1];
      };
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        entry(ai ^ 1) = fma(sx[j], kQ1.G[2 * j][ai][ai ^ 1], entry(ai ^ 1));
        entry(ai ^ 2) = fma(sy[j], kQ1.G[(j & 1) + 4 * (j >> 1)][ai][ai ^ 2], entry(ai ^ 2));
        entry(ai ^ 4) = fma(sz[j], kQ1.G[j][ai][ai ^ 4], entry(ai ^ 4));
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        entry(ai ^ 3) = fma(sxy[j], kQ1.G[4 * j][ai][ai ^ 3], entry(ai ^ 3));
        entry(ai ^ 5) = fma(sxz[j], kQ1.G[2 * j][ai][ai ^ 5], entry(ai ^ 5));
        entry(ai ^ 6) = fma(syz[j], kQ1.G[j][ai][ai ^ 6], entry(ai ^ 6));
      }
      entry(ai ^ 7) = fma(sxy[0] + sxy[1], kQ1.G[0][ai][ai ^ 7], entry(ai ^ 7));
      __builtin_amdgcn_sched_barrier(0);  // (an element's coefficients live at a time)
    }
}

// Sum of the off-diagonal entries of neighbour plane z: its three lines of three,
// then the lines (26 entries added one after the other round at nearly the size of
// the diagonal that they make up: values of 16^3 off by 4.5e-17 in the norm instead
// of 3.2e-17, the nonlinear Jacobian's by 4.9e-17 instead of 3.4e-17).
__device__ inline double plane_off(const double (&acc)[27], int z) {
  const double l0 = (acc[9 * z] + acc[9 * z + 1]) + acc[9 * z + 2];
  const double l1 = z == 1 ? acc[12] + acc[14] : (acc[9 * z + 3] + acc[9 * z + 4]) + acc[9 * z + 5];
  const double l2 = (acc[9 * z + 6] + acc[9 * z + 7]) + acc[9 * z + 8];
  return (l0 + l1) + l2;
}

// Whether any row of the wavefront has neighbours on the boundary.
__device__ inline bool near_boundary(int ii, int jj, int kk, int N) {
  return __ballot(ii <= 1 || jj <= 1 || kk <= 1 || ii >= N - 1 || jj >= N - 1 || kk >= N - 1) != 0;
}

// Entries T0 .. T1 - 1 of an interior row whose neighbour lies on the boundary
// become zero (near: near_boundary).
template <int T0, int T1>
__device__ inline void zero_edges(bool near, int ii, int jj, int kk, int N, double (&acc)[27]) {
  if (!near) return;
  auto edge = [&](int d, int i) { return d == 0 ? i == 1 : d == 2 ? i == N - 1 : false; };
#pragma unroll
  for (int t = T0; t < T1; ++t) {
    double v = acc[t];
    asm("" : "+v"(v));  // a select, not a branch around what v comes from
    acc[t] = ((int)edge(t % 3, ii) | (int)edge((t / 3) % 3, jj) | (int)edge(t / 9, kk)) ? 0.0 : v;
  }
}

// Ensemble assembly (Alg. "assembly" made atomic-free by row ownership): a
// workgroup owns a 4 x 2 x 4 block of nodes for all S samples (32 S lanes,
// one per row and sample, sample fastest).  It first evaluates the
// coefficient (times h/8) at the 8 Gauss points of each of the 5 x 3 x 5
// elements touching the block, once per element and sample, into LDS
// (153.6 KB for s = 32); then each (row, sample) lane of an interior row
// gathers its 8 elements from LDS in ascending element id and adds the element
// rows in that fixed order, so the sums are deterministic and the coefficient
// is evaluated 2.3 times per row instead of 8.  A wavefront holds whole sample
// ensembles of its rows, so every store of a matrix entry writes full
// 128-byte lines (s = 32: two FP64 lines, one FP32 line); split over
// workgroups of fewer samples, the partial lines of the FP32 copy alone took
// longer than the whole assembly does now.
// BND (fused multigrid set-up of this level): 0 none; 1 D^-1 in FP32 and
// the Gershgorin bound of the FP32 values; 2 D^-1 and the bound of the FP64
// values.  Each lane forms its row's sum_j |a_ij| / a_ii in ascending entry
// order in FP64 exactly as k_mg_diag_bound does, and the workgroup writes
// the maximum over its rows per sample to bpart[tile][s].
// ADV: the advection-diffusion operator D + alpha C instead (the linear part
// of the nonlinear problem's Jacobian, Eq. fenl_lin_sys with beta = 0):
// every element row also gets alpha (h^2/8) C_ab, C_ab = sum_q N_a (v.dN_b),
// summed over the elements for the 27 neighbours (advection_entries).
// Bound by its FP64 operations and its writes, which overlap only in part.  With
// the coefficient summed along columns, 38 operations an element and no
// boundary tests around them, FP64 values of 64^3, s = 16 take 231 us (396
// before; the writes alone 134), s = 32 447 (578; 269), 128^3, s = 32 with the
// FP32 copy 4.11 ms (4.65; 3.20).
// The body of k_assemble_tile for tile `bid`; xzero (nullable): a solution
// [n][s] whose rows of the tile are set to zero too.
template <int S, int BND, bool ADV>
__device__ __forceinline__ void assemble_tile_body(int N, const double* __restrict__ kl_sqrt_lam,
                                                   const int32_t* __restrict__ kl_triple,
                                                   const double* __restrict__ kl_phi, int M, double kappa0,
                                                   double sigma, double fsrc, double alpha, double vx, double vy,
                                                   double vz, const double* __restrict__ xi,
                                                   const int32_t* __restrict__ row_ptr, double* __restrict__ values,
                                                   float* __restrict__ values32, double* __restrict__ rhs,
                                                   void* __restrict__ dinv, double* __restrict__ bpart, int64_t bid,
                                                   double* __restrict__ xzero) {
  using T = AsmTile<32, 2>;
  constexpr int SB = S, NT = T::R * S;
  constexpr int TX = T::TX, TY = T::TY, EX = T::EX, EY = T::EY, NE = T::NE;
  constexpr int NTAB = tab_doubles<T::EX, T::EY, T::EZ>(kAsmMaxM);
  static_assert(NT <= NE * 8 * SB && NTAB >= 27, "tile shape");
  // [kappa at the Gauss points, [element][q][sample] | the tile's 1D KL
  // factors]; after the coefficients the factor area takes the advection
  // entries, after the row pass the kappa area the per-row bounds
  __shared__ double s_buf[NE * 8 * SB + NTAB];
  double* s_k = s_buf;
  double* s_tab = s_buf + NE * 8 * SB;
  double* s_adv = s_tab;
  const int n1 = N + 1;
  int64_t tile_id;
  int sg, x0, y0, z0;
  tile_decode<TX, TY, T::TZ, 1>(N, (uint32_t)bid, &tile_id, &sg, &x0, &y0, &z0);
  const int e0 = 0;
  const double h = 1.0 / (double)N;
  tile_coefficients<NT, SB, EX, EY, T::EZ>(N, kl_sqrt_lam, kl_triple, kl_phi, M, kappa0, sigma, xi, e0,
                                                  x0 - 1, y0 - 1, z0 - 1, h * 0.125, s_tab, s_k);
  if (ADV) {
    advection_entries(alpha * h * h, vx, vy, vz, s_adv);
    __syncthreads();
  }

  const int r = threadIdx.x / SB, sb = threadIdx.x % SB;
  const int rx = r % TX, ry = (r / TX) % TY, rz = r / (TX * TY);
  const int ii = x0 + rx, jj = y0 + ry, kk = z0 + rz;
  const bool live = ii <= N && jj <= N && kk <= N;
  if (!BND && !live) return;
  double qrow = 0.0;  // this row's Gershgorin ratio (BND)
  const int e = e0 + sb;
  if (live) {
    const int64_t row = (int64_t)ii + n1 * ((int64_t)jj + (int64_t)n1 * kk);
    const bool bnd_row = (ii == 0 || ii == N || jj == 0 || jj == N || kk == 0 || kk == N);
    const int64_t at = (int64_t)row_ptr[row] * S + e;
    // with 32 samples a wavefront's store covers whole 128-byte lines (FP32
    // and FP64), which then go out non-temporally (measured 4.98 -> 4.87 ms at
    // 128^3); smaller ensembles write partial lines, whose pieces are better
    // merged in L2 by ordinary stores
    constexpr bool NT = S == 32;
    auto st = [](auto* p, auto v) {
      if (NT) __builtin_nontemporal_store(v, p);
      else *p = v;
    };
    const bool near = near_boundary(ii, jj, kk, N);
    double dg = 1.0;
    if (bnd_row) {  // an identity row
      int k = 0;
      for (int t = 0; t < 27; ++t) {
        const int x = ii + t % 3 - 1, y = jj + (t / 3) % 3 - 1, z = kk + t / 9 - 1;
        if (x < 0 || y < 0 || z < 0 || x > N || y > N || z > N) continue;
        const double v = t == 13 ? 1.0 : 0.0;
        if (values) st(values + at + k * S, v);
        if (values32) st(values32 + at + k * S, (float)v);
        ++k;
      }
      qrow = 1.0;
    } else {
      double acc[27];
#pragma unroll
      for (int t = 0; t < 27; ++t) acc[t] = 0.0;
      diffusion_elements<T, SB, -1>(s_k, rx, ry, rz, sb, acc);
      diffusion_elements<T, SB, 0>(s_k, rx, ry, rz, sb, acc);
      // every element row sums to zero (the shape functions sum to one, so
      // sum_b grad N_b = 0, and C_ab = sum_q N_a v . grad N_b too), hence so
      // does the assembled row before the boundary conditions: its diagonal is
      // minus the sum of its other entries (plane_off), which saves the 8 diagonal element entries' Gauss sums
      if (ADV)
#pragma unroll
        for (int t = 0; t < 27; ++t)
          if (t != 13) acc[t] += s_adv[t];
      acc[13] = -((plane_off(acc, 0) + plane_off(acc, 1)) + plane_off(acc, 2));
      zero_edges<0, 27>(near, ii, jj, kk, N, acc);
      if (BND) {
        double sabs = 0.0;
#pragma unroll
        for (int t = 0; t < 27; ++t) {
          const double vc = BND == 1 ? (double)(float)acc[t] : acc[t];  // the value the cycle runs on
          sabs += fabs(vc);
          if (t == 13) dg = vc;
        }
        qrow = sabs / dg;
      }
      if (values)
#pragma unroll
        for (int t = 0; t < 27; ++t) st(values + at + t * S, acc[t]);
      if (values32)
#pragma unroll
        for (int t = 0; t < 27; ++t) st(values32 + at + t * S, (float)acc[t]);
    }
    st(rhs + row * S + e, bnd_row ? 0.0 : 8.0 * (fsrc * h * h * h * 0.125));  // of eight elements
    if (xzero) st(xzero + row * S + e, 0.0);
    if (BND == 1) st((float*)dinv + row * S + e, 1.0f / (float)dg);
    if (BND == 2) st((double*)dinv + row * S + e, 1.0 / dg);
  }
  if (BND) {
    __syncthreads();  // every lane is done with s_k
    double* s_q = s_k;
    s_q[threadIdx.x] = qrow;
    __syncthreads();
    if (threadIdx.x < SB) {
      double m = 0.0;
      for (int rr = 0; rr < T::R; ++rr) {
        const double q = s_q[rr * SB + threadIdx.x];
        m = q > m ? q : m;
      }
      bpart[tile_id * S + threadIdx.x] = m;
    }
  }
}

// Waves a SIMD that the tiles in LDS allow: the registers are cut to match.
template <int S>
constexpr int kAsmWaves = S >= 16 ? 4 : 3;

template <int S, int BND, bool ADV>
__global__ __launch_bounds__((32 * S), (kAsmWaves<S>)) void k_assemble_tile(int N, const double* __restrict__ kl_sqrt_lam,
                                                           const int32_t* __restrict__ kl_triple,
                                                           const double* __restrict__ kl_phi, int M, double kappa0,
                                                           double sigma, double fsrc, double alpha, double vx,
                                                           double vy, double vz, const double* __restrict__ xi,
                                                           const int32_t* __restrict__ row_ptr,
                                                           double* __restrict__ values, float* __restrict__ values32,
                                                           double* __restrict__ rhs, void* __restrict__ dinv,
                                                           double* __restrict__ bpart) {
  assemble_tile_body<S, BND, ADV>(N, kl_sqrt_lam, kl_triple, kl_phi, M, kappa0, sigma, fsrc, alpha, vx, vy, vz, xi,
                                  row_ptr, values, values32, rhs, dinv, bpart, blockIdx.x, nullptr);
}

// The assemblies of every group of a batch in one launch: workgroup b takes
// tile b - tile0 of group blk_grp[b] (FP64 values and load vector, the
// solution set to zero).
template <int S>
__global__ __launch_bounds__((32 * S), (kAsmWaves<S>)) void kb_assemble(const AsmGroupDev* __restrict__ groups,
                                                       const int32_t* __restrict__ blk_grp, int M, double kappa0,
                                                       double sigma, double fsrc) {
  const AsmGroupDev& g = groups[blk_grp[blockIdx.x]];
  assemble_tile_body<S, 0, false>(g.N, g.sq, g.tr, g.phi, M, kappa0, sigma, fsrc, 0.0, 0.0, 0.0, 0.0, g.xi, g.rp,
                                  g.values, nullptr, g.rhs, nullptr, nullptr, (int64_t)blockIdx.x - g.tile0, g.x);
}

// Residual and Jacobian of the nonlinear problem (Sec. 4, Eq.
// diffusion_sys, Eq. fenl_lin_sys, Alg. "assembly" with alpha, beta != 0),
// row-owned like k_assemble_tile (same tiling, the coefficient times h/8 kept
// in LDS per patch element).  The Jacobian's row a is
//   J_ab = D_ab + alpha (h^2/8) C_ab + 2 beta (h^3/8) R_ab, summed over the
//   elements, D_ab = (h/8) sum_q kappa_q G_q[a][b], C_ab = sum_q N_a (v.dN_b),
//   R_ab = sum_q u_q N_a N_b,
// u_q the interpolated solution at Gauss point q.  Since the diffusion and
// advection terms are linear in u and the reaction term quadratic, the
// residual is
//   F_a = sum_b (D_ab + alpha (h^2/8) C_ab + beta (h^3/8) R_ab) u_b
//         - (h^3/8) f sum_q N_a,
// so no gradient of u_h is formed.  Boundary rows (F = u, identity rows) need
// no element, and every other row has all eight, so only D takes a loop over
// them (its diagonal is minus the sum of the row's other linear entries, whose
// sum is zero as in k_assemble_tile).  C and R come for the 27 neighbours at
// once, as products over the axes of what the two elements of an axis add up
// to: C has the 1D mass (1/6, 2/3, 1/6) and first derivative (-1/2, 0, 1/2),
// the same for all rows; R contracts the 27 nodal values axis by axis with the
// 1D triple products sum_q l_a l_b l_c, 1/2 when a = b = c and 1/6 otherwise
// (reaction_line).  The nodal values of the tile and its rim are staged in LDS
// (the KL factors' area) once, on their way while the coefficient is summed.
// Boundary columns of interior rows are stored as zeros; load (optional) = the
// source part of F.
// Bound by the issue of its FP64 operations, about 1000 a row and sample: at
// 64^3, s = 16 F alone takes 236 us and F with the FP32 Jacobian 300 (451 and
// 510 with C and R summed element by element and the nodal values gathered from
// memory by every element).
//
// Reaction sums of one axis, times 6: from the values at the nodes -1, 0, 1
// those of the row's neighbours -1, 0, 1.
__device__ inline void reaction_line(double um, double u0, double up, double& rm, double& r0, double& rp) {
  rm = um + u0;
  rp = u0 + up;
  r0 = fma(u0, 4.0, rm + rp);
}

// What a tile holds in LDS beside the coefficient: its KL factors, then the
// nodal values of the tile and its rim and the 27 advection entries.
template <typename T, int SB>
__host__ __device__ constexpr int nl_tab_doubles() {
  constexpr int nodes = (T::TX + 2) * (T::TY + 2) * (T::TZ + 2) * SB + 27;
  constexpr int factors = tab_doubles<T::EX, T::EY, T::EZ>(kAsmMaxM);
  return nodes > factors ? nodes : factors;
}

// OUT: the Jacobian in FP64 (1), in FP32 (2), both (3), or F alone (0).
template <int S, int SB, int OUT>
__global__ __launch_bounds__((32 * SB), 3) void k_nl_assemble(int N, const double* __restrict__ kl_sqrt_lam,
                                                         const int32_t* __restrict__ kl_triple,
                                                         const double* __restrict__ kl_phi, int M, double kappa0,
                                                         double sigma, double fsrc, double alpha, double beta,
                                                         double vx, double vy, double vz, const double* __restrict__ xi,
                                                         const int32_t* __restrict__ row_ptr,
                                                         const double* __restrict__ u, double* __restrict__ values,
                                                         float* __restrict__ values32, double* __restrict__ F,
                                                         double* __restrict__ load) {
  using T = AsmTile<32, 2>;  // SB of the S samples of a 4 x 2 x 4 node block
  constexpr int NT = T::R * SB, G = S / SB;
  constexpr int TX = T::TX, TY = T::TY, TZ = T::TZ, EX = T::EX, EY = T::EY, NE = T::NE;
  constexpr int UX = TX + 2, UY = TY + 2, UZ = TZ + 2, NU = UX * UY * UZ * SB, LU = (NU + NT - 1) / NT;
  __shared__ double s_buf[NE * 8 * SB + nl_tab_doubles<T, SB>()];
  double* s_k = s_buf;
  double* s_tab = s_buf + NE * 8 * SB;
  double* s_u = s_tab;         // [z][y][x][sample]
  double* s_adv = s_tab + NU;  // advection entry of neighbour t
  int64_t tile_id;
  int sg, x0, y0, z0;
  tile_decode<TX, TY, TZ, G>(N, blockIdx.x, &tile_id, &sg, &x0, &y0, &z0);
  const int e0 = sg * SB;
  const int n1 = N + 1;
  const double h = 1.0 / (double)N;
  double un[LU];
#pragma unroll
  for (int i = 0; i < LU; ++i) {
    const int t = threadIdx.x + i * NT, node = t / SB;
    const int x = x0 - 1 + node % UX, y = y0 - 1 + (node / UX) % UY, z = z0 - 1 + node / (UX * UY);
    un[i] = t < NU && x >= 0 && y >= 0 && z >= 0 && x <= N && y <= N && z <= N
                ? u[((int64_t)x + n1 * ((int64_t)y + (int64_t)n1 * z)) * S + e0 + t % SB]
                : 0.0;
  }
  tile_coefficients<NT, SB, EX, EY, T::EZ>(N, kl_sqrt_lam, kl_triple, kl_phi, M, kappa0, sigma, xi, e0,
                                                  x0 - 1, y0 - 1, z0 - 1, h * 0.125, s_tab, s_k);
#pragma unroll
  for (int i = 0; i < LU; ++i)
    if (threadIdx.x + i * NT < NU) s_u[threadIdx.x + i * NT] = un[i];
  advection_entries(alpha * h * h, vx, vy, vz, s_adv);
  __syncthreads();

  const int rr = threadIdx.x / SB, sbl = threadIdx.x % SB;
  const int rx = rr % TX, ry = (rr / TX) % TY, rz = rr / (TX * TY);
  const int ii = x0 + rx, jj = y0 + ry, kk = z0 + rz;
  if (ii > N || jj > N || kk > N) return;
  const int e = e0 + sbl;
  const int64_t row = (int64_t)ii + n1 * ((int64_t)jj + (int64_t)n1 * kk);
  const bool bnd_row = (ii == 0 || ii == N || jj == 0 || jj == N || kk == 0 || kk == N);
  const int64_t at = OUT ? (int64_t)row_ptr[row] * S + e : 0;
  auto put = [&](int k, double v) {  // entry k of the row
    if (OUT & 1) values[at + k * S] = v;
    if (OUT & 2) values32[at + k * S] = (float)v;
  };
  const double* su = s_u + ((rz * UY + ry) * UX + rx) * SB + sbl;  // node (-1, -1, -1) of the row
  if (bnd_row) {
    if (OUT) {
      int k = 0;
      for (int t = 0; t < 27; ++t) {
        const int x = ii + t % 3 - 1, y = jj + (t / 3) % 3 - 1, z = kk + t / 9 - 1;
        if (x >= 0 && y >= 0 && z >= 0 && x <= N && y <= N && z <= N) put(k++, t == 13 ? 1.0 : 0.0);
      }
    }
    F[row * S + e] = u[row * S + e];
    if (load) load[row * S + e] = 0.0;
    return;
  }

  const double wr = h * h * h * 0.125;  // reaction and source: w_q
  const double wb = wr * beta / 216.0;  // the reaction sums are 6^3 times theirs
  const double la = 8.0 * (wr * fsrc);  // an element's load on a node, of eight
  double fa = 0.0, off = 0.0;
  double acc[27];
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = 0.0;
  // reaction sums of neighbour plane z over its own axes
  auto plane_sums = [&](int z, double* r) {
    double a[9];
#pragma unroll
    for (int y = 0; y < 3; ++y) {
      const double* p = su + (z * UY + y) * UX * SB;
      reaction_line(p[0], p[SB], p[2 * SB], a[3 * y], a[3 * y + 1], a[3 * y + 2]);
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) reaction_line(a[x], a[3 + x], a[6 + x], r[x], r[3 + x], r[6 + x]);
  };
  // entries of neighbour plane z from its linear ones and reaction sums; the
  // linear entries of a row sum to zero, so they take differences of u (fewer
  // digits cancel)
  const double u0 = su[((UY + 1) * UX + 1) * SB];
  auto finish_plane = [&](int z, const double* r) {
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      const int t = z * 9 + j;
      const double ut = su[((z * UY + j / 3) * UX + j % 3) * SB], rb = wb * r[j];
      if (t != 13) fa = fma(acc[t], ut - u0, fa);
      fa = fma(rb, ut, fa);
      acc[t] = fma(2.0, rb, acc[t]);
    }
    if (!OUT) return;
    if (z == 0) zero_edges<0, 9>(true, ii, jj, kk, N, acc);
    if (z == 1) zero_edges<9, 18>(true, ii, jj, kk, N, acc);
    if (z == 2) zero_edges<18, 27>(true, ii, jj, kk, N, acc);
#pragma unroll
    for (int j = 0; j < 9; ++j) put(z * 9 + j, acc[z * 9 + j]);
  };
  auto linear_plane = [&](int z) {  // advection; the off-diagonal sum
#pragma unroll
    for (int t = z * 9; t < z * 9 + 9; ++t)
      if (t != 13) acc[t] += s_adv[t];
    off += plane_off(acc, z);
  };

  // plane by plane, so that few accumulators are live: plane -1 is complete
  // after the lower elements
  double pm[9], p0[9], r[9];
  diffusion_elements<T, SB, -1>(s_k, rx, ry, rz, sbl, acc);
  plane_sums(0, pm);
  plane_sums(1, p0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    r[j] = pm[j] + p0[j];
    pm[j] = fma(p0[j], 4.0, r[j]);
  }
  linear_plane(0);
  finish_plane(0, r);
  __builtin_amdgcn_sched_barrier(0);
  diffusion_elements<T, SB, 0>(s_k, rx, ry, rz, sbl, acc);
  plane_sums(2, r);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    r[j] = p0[j] + r[j];
    p0[j] = pm[j] + r[j];
  }
  linear_plane(1);
  linear_plane(2);
  acc[13] = -off;
  finish_plane(1, p0);
  finish_plane(2, r);
  F[row * S + e] = fa - la;
  if (load) load[row * S + e] = la;
}

// Per-sample extremes of the coefficient over the 8 N^3 Gauss points of the
// mesh.  FP64 arithmetic bounds it, so the sum over the modes is contracted
// axis by axis: for one line of Gauss points along x (fixed y and z) the modes
// with the same x factor X_i collapse into one weight
//   W_i = sum over the modes m with x index i of c_m Y_m(y) Z_m(z),
// kappa = kappa0 + sum_i W_i X_i(x), and the 10 leading modes have 3 different
// x factors.  A lane owns a line; X_i(x) is the same for every lane of a
// wavefront and comes from scalar loads (16 operations and two NaN tests per
// point when every element summed its modes by itself; now 3.5).  A sample's lines are dealt to as many
// workgroups as fill the chip, whose extremes meet in 64-bit atomics on
// order-preserving keys (exact in any order).  512 samples at 64^3, 10 modes:
// 201 us, against 2432 us for one workgroup a sample.
// A coefficient that is NaN anywhere makes both extremes NaN.

// Bits of a double as an unsigned key of the same order.
__device__ inline unsigned long long ext_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return b >> 63 ? ~b : b | 0x8000000000000000ull;
}
__device__ inline double ext_value(unsigned long long k) {
  return __longlong_as_double((long long)(k >> 63 ? k & 0x7fffffffffffffffull : ~k));
}
// Keys beyond every number's, so that they win: NaN in the minimum's and in
// the maximum's array.
constexpr unsigned long long kExtNanLo = 0ull, kExtNanHi = ~0ull;

__global__ void k_kl_extrema_keys(int64_t s, unsigned long long* __restrict__ lo, unsigned long long* __restrict__ hi) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= s) return;
  lo[e] = ext_key(INFINITY);
  hi[e] = ext_key(-INFINITY);
}

__global__ void k_kl_extrema_values(int64_t s, double* __restrict__ kmin, double* __restrict__ kmax) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= s) return;
  const unsigned long long l = (unsigned long long)__double_as_longlong(kmin[e]),
                           h = (unsigned long long)__double_as_longlong(kmax[e]);
  kmin[e] = l == kExtNanLo ? NAN : ext_value(l);
  kmax[e] = h == kExtNanHi ? NAN : ext_value(h);
}

// Extremes along one line.  The 1D modes are even (index 0, 2, ...) or odd
// about the middle of the axis and the Gauss points mirror there, so the
// coefficient at a point and at its mirror image is E + O and E - O of the
// even and the odd part: a pair costs its multiply-adds once, E - |O| and
// E + |O| (measured 293 -> 201 us).  The extremes are those of the modes' sum:
// kappa0 is added to them afterwards, one rounding at its size (with E starting
// from kappa0 there was one a mode index, and twice the error).  With CHECK, NaN
// is looked for.
template <int NX, bool CHECK>
__device__ inline void line_extrema(const double* __restrict__ phi, int two_n, const double* w, double& lo,
                                    double& hi, int& bad) {
#pragma unroll 8
  for (int x = 0; x < two_n / 2; ++x) {
    double ev = w[0] * phi[x], od = 0.0;
#pragma unroll
    for (int i = 2; i < NX; i += 2) ev = fma(w[i], phi[i * (int64_t)two_n + x], ev);
#pragma unroll
    for (int i = 1; i < NX; i += 2) od = fma(w[i], phi[i * (int64_t)two_n + x], od);
    const double l = ev - fabs(od), h = ev + fabs(od);
    if (CHECK) bad |= (l != l) | (h != h);
    lo = fmin(lo, l);
    hi = fmax(hi, h);
  }
}

// The lines of one workgroup: every step-th from line0 (one a lane).
template <int NX>
__device__ inline void lines_extrema(int two_n, int64_t line0, int64_t step, const int32_t* __restrict__ kl_triple,
                                     const double* __restrict__ kl_phi, const double* s_cm, int M, double& lo,
                                     double& hi, int& bad) {
  const int64_t lines = (int64_t)two_n * two_n;
  for (int64_t l = line0; l < lines; l += step) {
    const int y = (int)(l % two_n), z = (int)(l / two_n);
    double w[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) w[i] = 0.0;
    for (int m = 0; m < M; ++m) {
      const int ix = kl_triple[3 * m];
      const double v = s_cm[m] * (kl_phi[kl_triple[3 * m + 1] * (int64_t)two_n + y] *
                                  kl_phi[kl_triple[3 * m + 2] * (int64_t)two_n + z]);
#pragma unroll
      for (int i = 0; i < NX; ++i) w[i] += i == ix ? v : 0.0;
    }
    // weights this small cannot overflow at a point, so no point is NaN
    bool plain = true;
#pragma unroll
    for (int i = 0; i < NX; ++i) plain = plain && fabs(w[i]) < 1e290;
    if (plain) line_extrema<NX, false>(kl_phi, two_n, w, lo, hi, bad);
    else line_extrema<NX, true>(kl_phi, two_n, w, lo, hi, bad);
  }
}

__global__ __launch_bounds__(256) void k_kl_extrema(int N, const double* __restrict__ kl_sqrt_lam,
                                                     const int32_t* __restrict__ kl_triple,
                                                     const double* __restrict__ kl_phi, int M, double kappa0,
                                                     double sigma, const double* __restrict__ xi,
                                                     unsigned long long* __restrict__ klo,
                                                     unsigned long long* __restrict__ khi) {
  __shared__ double s_cm[kAsmMaxM];
  __shared__ double s_lo[4], s_hi[4];
  __shared__ int s_bad[4];
  const int64_t e = blockIdx.y;
  if (threadIdx.x < M) s_cm[threadIdx.x] = sigma * kl_sqrt_lam[threadIdx.x] * xi[e * M + threadIdx.x];
  // The x indices of the leading modes are 0 .. nx - 1.  Mode (i, 0, 0) comes
  // after all permutations of (j, 0, 0), j < i, and after (0, 0, i) and (0, i, 0), so
  // index i takes 3 i + 1 modes: kAsmMaxM hold at most 6, and no row of the table
  // past nx (at most M) is read.
  static_assert(kAsmMaxM < 3 * 6 + 1, "x indices up to 5");
  int nx = 1;
  for (int m = 0; m < M; ++m) nx = kl_triple[3 * m] >= nx ? kl_triple[3 * m] + 1 : nx;
  __syncthreads();
  double lo = INFINITY, hi = -INFINITY;
  int bad = 0;
  const int64_t l0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  const int two_n = 2 * N;
  if (M > 0) switch (nx) {
      case 1: lines_extrema<1>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
      case 2: lines_extrema<2>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
      case 3: lines_extrema<3>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
      case 4: lines_extrema<4>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
      case 5: lines_extrema<5>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
      default: lines_extrema<6>(two_n, l0, step, kl_triple, kl_phi, s_cm, M, lo, hi, bad); break;
    }
  else lo = hi = 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
    bad |= __shfl_xor(bad, off, 64);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
    s_bad[wave] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int v = 1; v < 4; ++v) {
      lo = fmin(lo, s_lo[v]);
      hi = fmax(hi, s_hi[v]);
      bad |= s_bad[v];
    }
    lo += kappa0;  // (every workgroup has a line, so both are a point's)
    hi += kappa0;
    bad |= (lo != lo) | (hi != hi);
    if (gridDim.x == 1) {  // a sample's only workgroup: the values themselves
      ((double*)klo)[e] = bad ? NAN : lo;
      ((double*)khi)[e] = bad ? NAN : hi;
    } else {
      atomicMin(klo + e, bad ? kExtNanLo : ext_key(lo));
      atomicMax(khi + e, bad ? kExtNanHi : ext_key(hi));
    }
  }
}

template <int R, int TY>
static int64_t tiles_of(int N) {
  using T = AsmTile<R, TY>;
  return (int64_t)((N + T::TX) / T::TX) * ((N + T::TY) / T::TY) * ((N + T::TZ) / T::TZ);
}

// Samples per workgroup of the nonlinear assembly: 8 (256 lanes, 3 per CU;
// at 128^3, s = 32 this ran 7.9 ms per launch against 8.1 ms for all 32
// samples in one workgroup, whose full-line stores do not pay for its
// single workgroup per CU in this arithmetic-bound kernel).
static constexpr int nl_sb(int S) { return S < 8 ? S : 8; }

// Tiles of both assemblies (rows of the linear one's fused bound partials).
int64_t asm_tiles(int N, int S) {
  (void)S;
  return tiles_of<32, 2>(N);
}

ens_status batch_assemble_launch(int S, const AsmGroupDev* groups, const int32_t* blk_grp, int64_t blocks,
                                 const ens_problem& prob, hipStream_t st) {
  if (blocks <= 0) return ENS_OK;
  switch (S) {
#define ENS_BASM(SS)                                                                                         \
  case SS:                                                                                                   \
    hipLaunchKernelGGL(kb_assemble<SS>, dim3((unsigned)blocks), dim3(32 * SS), 0, st, groups, blk_grp, prob.M, \
                       prob.kappa0, prob.sigma, prob.f);                                                     \
    break;
    ENS_BASM(8)
    ENS_BASM(16)
    ENS_BASM(32)
#undef ENS_BASM
    default:
      set_error("batch ensemble size %d not compiled in (8, 16, 32)", S);
      return ENS_E_UNSUPPORTED;
  }
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status assemble_launch(int N, const ens_graph* graph, const double* sq, const int32_t* tr, const double* phi,
                           const ens_problem* prob, int s, const double* xi, double* values, float* values32,
                           double* rhs, int bnd, void* dinv, double* bpart, hipStream_t stream, const double* adv) {
  int64_t n = 0, nnz = 0;
  ens_status st = ens_mesh_sizes(N, &n, &nnz, nullptr);
  if (st != ENS_OK) return st;
  const bool with_adv = adv && adv[0] != 0.0;
  if (with_adv && bnd == 0) {
    set_error("the advection-diffusion assembly is built only with a fused multigrid set-up");
    return ENS_E_UNSUPPORTED;
  }
  const double av[4] = {with_adv ? adv[0] : 0.0, with_adv ? adv[1] : 0.0, with_adv ? adv[2] : 0.0,
                        with_adv ? adv[3] : 0.0};
  const int M = prob->M;
  prof_begin(ENS_K_ASSEMBLE, stream);
  switch (s) {
#define ENS_ASM_LAUNCH(SS, BB, AA)                                                                                \
  hipLaunchKernelGGL((k_assemble_tile<SS, BB, AA>), dim3((unsigned)asm_tiles(N, SS)), dim3(32 * SS), 0, stream, N, sq, \
                     tr, phi, M, prob->kappa0, prob->sigma, prob->f, av[0], av[1], av[2], av[3], xi, graph->row_ptr,  \
                     values, values32, rhs, dinv, bpart)
#define ENS_ASM_CASE(SS)                                         \
  case SS:                                                       \
    if (with_adv && bnd == 1) ENS_ASM_LAUNCH(SS, 1, true);       \
    else if (with_adv && bnd == 2) ENS_ASM_LAUNCH(SS, 2, true);  \
    else if (bnd == 1) ENS_ASM_LAUNCH(SS, 1, false);             \
    else if (bnd == 2) ENS_ASM_LAUNCH(SS, 2, false);             \
    else ENS_ASM_LAUNCH(SS, 0, false);                           \
    break;
    ENS_ASM_CASE(4)
    ENS_ASM_CASE(8)
    ENS_ASM_CASE(16)
    ENS_ASM_CASE(32)
#undef ENS_ASM_CASE
#undef ENS_ASM_LAUNCH
  }
  ENS_LAUNCH_CHECK();
  double bytes = (double)nnz * s * ((values ? 8.0 : 0.0) + (values32 ? 4.0 : 0.0)) + (double)n * s * 8.0 + 4.0 * (n + 1);
  if (bnd) bytes += (double)n * s * (bnd == 1 ? 4.0 : 8.0);
  prof_end(ENS_K_ASSEMBLE, stream, bytes);
  return ENS_OK;
}

// The KL table's parts (layout of ens_kl_build).
void kl_parts(const void* kl, int M, const double** sq, const int32_t** tr, const double** phi) {
  const char* base = (const char*)kl;
  const size_t phi_off = ((size_t)M * 5 * sizeof(double) + (size_t)M * 4 * sizeof(int32_t) + 15) & ~(size_t)15;
  *sq = (const double*)base;
  *tr = (const int32_t*)(base + (size_t)M * 5 * sizeof(double) + (size_t)M * sizeof(int32_t));
  *phi = (const double*)(base + phi_off);
}

}  // namespace ens

using namespace ens;

extern "C" ens_status ens_assemble(int32_t N, const ens_graph* graph, const void* kl, const ens_problem* prob,
                                   int32_t s, const double* xi, double* values, float* values32, double* rhs,
                                   hipStream_t stream) {
  int64_t n = 0, nnz = 0;
  ens_status st = ens_mesh_sizes(N, &n, &nnz, nullptr);
  if (st != ENS_OK) return st;
  ENS_ARG_CHECK(graph && prob, "null graph or problem");
  ENS_ARG_CHECK(graph->n == n && graph->nnz == nnz && graph->row_ptr && graph->col_idx,
                "graph does not match the mesh");
  ENS_ARG_CHECK(values && rhs, "null output");
  ENS_ARG_CHECK(prob->M >= 0 && prob->M <= kAsmMaxM, "M out of range");
  ENS_ARG_CHECK(prob->M == 0 || (kl && xi), "null KL table or inputs");
  if (!supported_s(s)) {
    set_error("ensemble size %d not compiled in", s);
    return ENS_E_UNSUPPORTED;
  }
  const double *sq = nullptr, *phi = nullptr;
  const int32_t* tr = nullptr;
  kl_parts(kl, prob->M, &sq, &tr, &phi);
  return assemble_launch(N, graph, sq, tr, phi, prob, s, xi, values, values32, rhs, 0, nullptr, nullptr, stream,
                         nullptr);
}

extern "C" ens_status ens_nl_assemble(int32_t N, const ens_graph* graph, const void* kl,
                                      const ens_nl_problem* prob, int32_t s, const double* xi, const double* u,
                                      double* values, float* values32, double* F, double* load,
                                      hipStream_t stream) {
  int64_t n = 0, nnz = 0;
  ens_status st = ens_mesh_sizes(N, &n, &nnz, nullptr);
  if (st != ENS_OK) return st;
  ENS_ARG_CHECK(graph && prob, "null graph or problem");
  ENS_ARG_CHECK(graph->n == n && graph->nnz == nnz && graph->row_ptr && graph->col_idx,
                "graph does not match the mesh");
  ENS_ARG_CHECK(u && F, "null u or F");
  ENS_ARG_CHECK(prob->M >= 0 && prob->M <= kAsmMaxM, "M out of range");
  ENS_ARG_CHECK(prob->M == 0 || (kl && xi), "null KL table or inputs");
  if (!supported_s(s)) {
    set_error("ensemble size %d not compiled in", s);
    return ENS_E_UNSUPPORTED;
  }
  const int M = prob->M;
  const double *sq, *phi;
  const int32_t* tr;
  kl_parts(kl, M, &sq, &tr, &phi);
  prof_begin(ENS_K_NL_ASSEMBLE, stream);
  switch (s) {
#define ENS_NL_LAUNCH(SS, JJ)                                                                                    \
  hipLaunchKernelGGL((k_nl_assemble<SS, nl_sb(SS), JJ>), dim3((unsigned)(asm_tiles(N, SS) * (SS / nl_sb(SS)))),      \
                     dim3(32 * nl_sb(SS)), 0, stream, N, sq, tr,                                                      \
                     phi, M, prob->kappa0, prob->sigma, prob->f, prob->alpha, prob->beta, prob->vx, prob->vy,       \
                     prob->vz, xi, graph->row_ptr, u, values, values32, F, load)
#define ENS_NL_CASE(SS)                                  \
  case SS:                                               \
    if (values && values32) ENS_NL_LAUNCH(SS, 3);        \
    else if (values32) ENS_NL_LAUNCH(SS, 2);             \
    else if (values) ENS_NL_LAUNCH(SS, 1);               \
    else ENS_NL_LAUNCH(SS, 0);                           \
    break;
    ENS_NL_CASE(4)
    ENS_NL_CASE(8)
    ENS_NL_CASE(16)
    ENS_NL_CASE(32)
#undef ENS_NL_CASE
#undef ENS_NL_LAUNCH
  }
  ENS_LAUNCH_CHECK();
  const double bytes = (values ? (double)nnz * s * 8.0 : 0.0) + (values32 ? (double)nnz * s * 4.0 : 0.0) +
                       (double)n * s * 8.0 * (load ? 3.0 : 2.0) + 4.0 * (n + 1);
  prof_end(ENS_K_NL_ASSEMBLE, stream, bytes);
  return ENS_OK;
}

extern "C" ens_status ens_kl_extrema(int32_t N, const void* kl, const ens_problem* prob, int32_t s,
                                     const double* xi, double* kmin, double* kmax, hipStream_t stream) {
  ENS_ARG_CHECK(N >= 1 && N <= 1024, "N out of range");
  ENS_ARG_CHECK(prob && s >= 1, "null problem or no samples");
  ENS_ARG_CHECK(prob->M >= 0 && prob->M <= kAsmMaxM, "M out of range");
  ENS_ARG_CHECK(prob->M == 0 || (kl && xi), "null KL table or inputs");
  ENS_ARG_CHECK(kmin && kmax, "null output");
  const double *sq = nullptr, *phi = nullptr;
  const int32_t* tr = nullptr;
  kl_parts(kl, prob->M, &sq, &tr, &phi);
  // enough workgroups a sample to fill the chip eight times over (or all of
  // its lines at once); the second grid dimension holds up to 65535 samples.
  // A sample of up to 1024 lines (16^3) has one, which needs no keys: one launch
  // instead of three, 10.4 us against 15.7 (20^3, in four more rounds, 16.2 both
  // ways).
  const int64_t lines = 4 * (int64_t)N * N, most = (lines + 255) / 256;
  int64_t per = (2048 + s - 1) / s;
  if (per > most) per = most;
  if (lines <= 1024) per = 1;
  const unsigned sb = (unsigned)(((int64_t)s + 255) / 256);
  if (per > 1)
    hipLaunchKernelGGL(k_kl_extrema_keys, dim3(sb), dim3(256), 0, stream, (int64_t)s, (unsigned long long*)kmin,
                       (unsigned long long*)kmax);
  for (int64_t e0 = 0; e0 < s; e0 += 65535) {
    const int64_t ne = s - e0 < 65535 ? s - e0 : 65535;
    hipLaunchKernelGGL(k_kl_extrema, dim3((unsigned)per, (unsigned)ne), dim3(256), 0, stream, N, sq, tr, phi, prob->M,
                       prob->kappa0, prob->sigma, xi + e0 * prob->M, (unsigned long long*)kmin + e0,
                       (unsigned long long*)kmax + e0);
  }
  if (per > 1) hipLaunchKernelGGL(k_kl_extrema_values, dim3(sb), dim3(256), 0, stream, (int64_t)s, kmin, kmax);
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}
