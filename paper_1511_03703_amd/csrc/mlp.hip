// Learned initial guess, network part: a 10 -> 256 -> 256 -> 32 MLP with
// GELU activations that maps the KL inputs y of a sample to the
// coefficients of a POD basis; its prediction only seeds CG.
//
// All matrix products run on gfx950 matrix cores (v_mfma_f32_16x16x32_bf16):
// BF16 operands, FP32 accumulation.  Bias, GELU, loss and Adam are FP32 on
// FP32 master weights.  Every product is written as one "NT" form,
//     C[m][n] = sum_k A[m][k] B[n][k]      (both operands K-contiguous),
// so each lane takes its 8-element MFMA fragment with one 16-byte load.
//
// The network is small (76,832 parameters), so a step is bound by the chain
// of its launches, not by its 0.12 GFLOP at a batch of 256.  A training step
// is two launches: k_mlp_rows takes 16 rows of the batch through the whole
// forward and backward pass (every product of it is local to the rows;
// activations pass between the layers in LDS) and k_mlp_update forms the
// weight gradients over the batch, each 16 x 16 tile by one wavefront, and
// takes the Adam step on them where they are.  Measured at a batch of 256:
// 21.3 us a step, against 98 us for 15 launches of one product or
// elementwise pass each.  Every product adds its K chunks of 32 in ascending
// order and every bias sum its rows in a fixed order, whatever the batch is
// split into.
//
// GELU is the exact form 0.5 z (1 + erf(z / sqrt 2)), derivative
// Phi(z) + z phi(z).
#include "common.hpp"

namespace ens {

constexpr int kIn = 10, kInPad = 32, kHid = 256, kOut = 32;
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kHid * kIn, kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid,
                  kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kOut * kHid, kParams = kOffB3 + kOut;

typedef uint16_t bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round-to-nearest-even FP32 -> BF16 (bit pattern)
__device__ inline bf16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
__device__ inline float from_bf16(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// 2 Phi(z) = 1 + erf(z / sqrt 2), which GELU and its derivative share.
__device__ inline float two_phi(float z) { return 1.0f + erff(z * 0.70710678118654752f); }
__device__ inline float gelu(float z, float p2) { return 0.5f * z * p2; }
__device__ inline float gelu_grad(float z, float p2) {
  return fmaf(z * 0.39894228040143268f, expf(-0.5f * z * z), 0.5f * p2);
}

// BF16 copies of the weights: W1 [256][32] (K padded), W2 and W2^T, W3 and W3^T.
__global__ void k_mlp_weights(const float* __restrict__ p, bf16_t* __restrict__ w1, bf16_t* __restrict__ w2,
                              bf16_t* __restrict__ w2t, bf16_t* __restrict__ w3, bf16_t* __restrict__ w3t) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < kHid * kInPad) {
    const int n = t / kInPad, k = t % kInPad;
    w1[t] = k < kIn ? to_bf16(p[kOffW1 + n * kIn + k]) : (bf16_t)0;
  }
  if (t < kHid * kHid) {
    const int n = t / kHid, k = t % kHid;
    const bf16_t v = to_bf16(p[kOffW2 + t]);
    w2[t] = v;
    w2t[k * kHid + n] = v;
  }
  if (t < kOut * kHid) {
    const int n = t / kHid, k = t % kHid;
    const bf16_t v = to_bf16(p[kOffW3 + t]);
    w3[t] = v;
    w3t[k * kOut + n] = v;
  }
}

// One Adam step (Kingma and Ba 2015, Algorithm 1) per element, FP32:
// moving averages of g and g^2, divided by the bias corrections c1 = 1 - b1^t
// and c2 = 1 - b2^t, eps added to the square root of the second moment.
// omb1 = 1 - b1 and omb2 = 1 - b2 come in as arguments, each the FP32
// rounding of the exact value (1.0f - 0.999f would carry the 1.3e-5 relative
// error of 0.999f into every second moment).
struct AdamStep {
  float lr, b1, b2, omb1, omb2, eps, c1, c2;
};

__device__ inline void adam_element(float& p, float g, float& m, float& v, const AdamStep& k) {
  m = fmaf(k.omb1, g, k.b1 * m);  // the contractions spelt out: every kernel rounds alike
  v = fmaf(g, k.omb2 * g, k.b2 * v);
  p -= k.lr * (m / k.c1) / (sqrtf(v / k.c2) + k.eps);
}

__global__ void k_adam(int64_t P, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, AdamStep k) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  adam_element(p[i], g[i], m[i], v[i], k);
}

// Bias corrections 1 - beta^t of step t = 1, 2, ... for beta = (0.9, 0.999);
// the powers are the products of the steps in order, carried from step to
// step.  1 - beta and 1 - beta^t are formed in FP64 from the decimal betas
// and rounded once to FP32.
struct AdamPowers {
  double p1 = 1.0, p2 = 1.0;
  void advance(int steps) {
    for (int k = 0; k < steps; ++k) {
      p1 *= 0.9;
      p2 *= 0.999;
    }
  }
  AdamStep step(float lr) const {
    return AdamStep{lr,    (float)0.9, (float)0.999,      (float)(1.0 - 0.9), (float)(1.0 - 0.999),
                    1e-8f, (float)(1.0 - p1), (float)(1.0 - p2)};
  }
};

// ------------------------------------------------------ the fused kernels ---

struct MlpWork {
  // transposed BF16 activations and gradients, [unit][batch]: the operands of
  // the weight gradients
  bf16_t *xt, *h1t, *h2t, *dyt, *dz2t, *dz1t;
  bf16_t *w1, *w2, *w2t, *w3, *w3t;
  float *dy, *dz2, *dz1;  // [batch][unit] FP32, summed into the bias gradients
  double* lossp;          // squared error of each 16 rows
};

constexpr int kRows = 16;            // batch rows of one k_mlp_rows workgroup
constexpr int kLdH = kHid + 8;       // LDS row of an activation tile: 16-byte aligned, rows on different banks
constexpr int kLdY = kOut + 8;

typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

__device__ inline f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Inputs k0 .. k0 + 7 of an FP32 row as a BF16 fragment, zero past its end.
__device__ inline bf16x8 input_frag(const float* __restrict__ row, int k0) {
  u16x8 u;
#pragma unroll
  for (int j = 0; j < 8; ++j) u[j] = k0 + j < kIn ? to_bf16(row[k0 + j]) : (uint16_t)0;
  return __builtin_bit_cast(bf16x8, u);
}

// 16 rows of the batch through the network, 16 wavefronts, each on 16 units
// (columns) of every layer; with TRAIN also the backward pass of the mean
// squared error down to the pre-activation gradients.  MFMA 16x16x32
// fragments: lane l holds A[l%16][8(l/16) .. 8(l/16)+7] and B[8(l/16) ..
// +7][l%16]; the result leaves D[4(l/16)+t][l%16], t = 0..3, in lane l, which
// is also how it holds the layer's pre-activations until the backward pass
// needs them.  The time is the chain of five products and their barriers;
// the weights (0.3 MB, from L2) do not depend on it, so their fragments are
// loaded ahead.  Reading the weights in FP32 and rounding them here, which
// would spare a forward pass the launch of k_mlp_weights, took 28 us longer:
// a lane's eight dwords are eight loads that touch 64 lines each.
template <bool TRAIN>
__global__ __launch_bounds__(1024) void k_mlp_rows(int B, const float* __restrict__ p, const float* __restrict__ xi,
                                                   const float* __restrict__ tgt, const int32_t* __restrict__ idx,
                                                   MlpWork w, float* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) bf16_t s_h1[kRows * kLdH];
  __shared__ __attribute__((aligned(16))) bf16_t s_h2[kRows * kLdH];
  __shared__ __attribute__((aligned(16))) bf16_t s_dy[kRows * kLdY];
  __shared__ double s_loss[2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4, n = 16 * wave + r, m0 = blockIdx.x * kRows;
  const int src = idx ? idx[m0 + r] : m0 + r;
  const bf16x8 xa = input_frag(xi + (int64_t)src * kIn, 8 * q);
  const bf16x8 w1f = *(const bf16x8*)(w.w1 + n * kInPad + 8 * q);
  bf16x8 w2f[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) w2f[k] = *(const bf16x8*)(w.w2 + n * kHid + 32 * k + 8 * q);
  const float b1 = p[kOffB1 + n], b2 = p[kOffB2 + n];

  f32x4 z1 = mfma_bf16(xa, w1f, (f32x4)0.0f), phi1, phi2;
  {
    u16x4 h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      z1[t] = z1[t] + b1;
      phi1[t] = two_phi(z1[t]);
      h[t] = to_bf16(gelu(z1[t], phi1[t]));
      s_h1[(4 * q + t) * kLdH + n] = h[t];
    }
    if (TRAIN) {
      *(u16x4*)(w.h1t + (int64_t)n * B + m0 + 4 * q) = h;
      if (wave == 0) {
        const u16x8 xu = __builtin_bit_cast(u16x8, xa);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (8 * q + j < kIn) w.xt[(int64_t)(8 * q + j) * B + m0 + r] = xu[j];
      }
    }
  }
  __syncthreads();

  f32x4 z2 = (f32x4)0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) z2 = mfma_bf16(*(const bf16x8*)(s_h1 + r * kLdH + 32 * k + 8 * q), w2f[k], z2);
  {
    u16x4 h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      z2[t] = z2[t] + b2;
      phi2[t] = two_phi(z2[t]);
      h[t] = to_bf16(gelu(z2[t], phi2[t]));
      s_h2[(4 * q + t) * kLdH + n] = h[t];
    }
    if (TRAIN) *(u16x4*)(w.h2t + (int64_t)n * B + m0 + 4 * q) = h;
  }
  bf16x8 w3f[8], w3tf, w2tf[8];
  float tg[4];
  if (wave < kOut / 16) {
#pragma unroll
    for (int k = 0; k < 8; ++k) w3f[k] = *(const bf16x8*)(w.w3 + n * kHid + 32 * k + 8 * q);
    if (TRAIN) {
#pragma unroll
      for (int t = 0; t < 4; ++t) tg[t] = tgt[(int64_t)(idx ? idx[m0 + 4 * q + t] : m0 + 4 * q + t) * kOut + n];
    }
  }
  if (TRAIN) {
    w3tf = *(const bf16x8*)(w.w3t + n * kOut + 8 * q);
#pragma unroll
    for (int k = 0; k < 8; ++k) w2tf[k] = *(const bf16x8*)(w.w2t + n * kHid + 32 * k + 8 * q);
  }
  __syncthreads();

  if (wave < kOut / 16) {
    f32x4 y = (f32x4)0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) y = mfma_bf16(*(const bf16x8*)(s_h2 + r * kLdH + 32 * k + 8 * q), w3f[k], y);
    const float b3 = p[kOffB3 + n];
    const float sc = 2.0f / (float)(B * kOut);
    double sq = 0.0;
    u16x4 h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int m = 4 * q + t;
      const float yv = y[t] + b3;
      if (out) out[(int64_t)(m0 + m) * kOut + n] = yv;
      if (TRAIN) {
        const float d = yv - tg[t];
        sq += (double)d * (double)d;
        const float g = sc * d;
        w.dy[(int64_t)(m0 + m) * kOut + n] = g;
        h[t] = to_bf16(g);
        s_dy[m * kLdY + n] = h[t];
      }
    }
    if (TRAIN) {
      *(u16x4*)(w.dyt + (int64_t)n * B + m0 + 4 * q) = h;
      sq = wave_sum_stride<1>(sq);
      if (lane == 0) s_loss[wave] = sq;
    }
  }
  if (!TRAIN) return;
  __syncthreads();
  if (threadIdx.x == 0) w.lossp[blockIdx.x] = s_loss[0] + s_loss[1];

  // dZ2 = (dY W3) GELU'(Z2), its BF16 tile in place of H1
  f32x4 dz = mfma_bf16(*(const bf16x8*)(s_dy + r * kLdY + 8 * q), w3tf, (f32x4)0.0f);
  {
    u16x4 h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float g = dz[t] * gelu_grad(z2[t], phi2[t]);
      w.dz2[(int64_t)(m0 + 4 * q + t) * kHid + n] = g;
      h[t] = to_bf16(g);
      s_h1[(4 * q + t) * kLdH + n] = h[t];
    }
    *(u16x4*)(w.dz2t + (int64_t)n * B + m0 + 4 * q) = h;
  }
  __syncthreads();

  // dZ1 = (dZ2 W2) GELU'(Z1)
  dz = (f32x4)0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) dz = mfma_bf16(*(const bf16x8*)(s_h1 + r * kLdH + 32 * k + 8 * q), w2tf[k], dz);
  {
    u16x4 h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float g = dz[t] * gelu_grad(z1[t], phi1[t]);
      w.dz1[(int64_t)(m0 + 4 * q + t) * kHid + n] = g;
      h[t] = to_bf16(g);
    }
    *(u16x4*)(w.dz1t + (int64_t)n * B + m0 + 4 * q) = h;
  }
}

// Workgroups of k_mlp_update: the 16 x 16 tiles of dW2, dW3 and dW1 (four a
// workgroup, one per wavefront), 16 bias columns each, and the loss.
constexpr int kTilesW2 = 256, kTilesW3 = 32, kTilesW1 = 16;
constexpr int kTileBlocks = (kTilesW2 + kTilesW3 + kTilesW1) / 4;
constexpr int kBiasBlocks = (kHid + kHid + kOut) / 16;
constexpr int kUpdateBlocks = kTileBlocks + kBiasBlocks + 1;

// The gradients of a batch whose rows k_mlp_rows took, each formed by the
// lane that owns the parameter: stored to grad, or (ADAM) used for the
// parameter's Adam step at once, the BF16 copies of the weights refreshed
// beside it, so neither the gradient nor the old copies cross a launch.
//   dW3[n][k] = sum_b dY[b][n] H2[b][k], dW2 and dW1 likewise;
//   db[n] = the column sums of dZ1, dZ2, dY in FP32: sixteen running sums over
//   the rows of equal b mod 16, combined in a fixed order.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_update(int B, MlpWork w, float* __restrict__ p, float* __restrict__ am,
                                                    float* __restrict__ av, AdamStep ad, float* __restrict__ grad,
                                                    float* __restrict__ loss) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int blk = blockIdx.x;
  if (blk < kTileBlocks) {
    const int r = lane & 15, q = lane >> 4;
    int t = blk * 4 + wave, nt, kt, ldw, cols;
    const bf16_t *a, *b;
    int64_t off;
    bf16_t *wc, *wt;
    int ldc, ldt;
    if (t < kTilesW2) {
      nt = t >> 4, kt = t & 15, ldw = kHid, cols = kHid, off = kOffW2;
      a = w.dz2t, b = w.h1t, wc = w.w2, wt = w.w2t, ldc = kHid, ldt = kHid;
    } else if (t < kTilesW2 + kTilesW3) {
      t -= kTilesW2;
      nt = t >> 4, kt = t & 15, ldw = kHid, cols = kHid, off = kOffW3;
      a = w.dyt, b = w.h2t, wc = w.w3, wt = w.w3t, ldc = kHid, ldt = kOut;
    } else {
      nt = t - kTilesW2 - kTilesW3, kt = 0, ldw = kIn, cols = kIn, off = kOffW1;
      a = w.dz1t, b = w.xt, wc = w.w1, wt = nullptr, ldc = kInPad, ldt = 0;
    }
    const int k = 16 * kt + r;
    const bf16_t* ar = a + (int64_t)(16 * nt + r) * B + 8 * q;
    const bf16_t* br = b + (int64_t)(k < cols ? k : 0) * B + 8 * q;
    const int64_t i0 = off + (int64_t)(16 * nt + 4 * q) * ldw + k;
    // the parameters and moments do not depend on the gradient: on their way
    // while it is formed
    float pv[4], mv[4], vv[4];
    if (ADAM && k < cols) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = i0 + (int64_t)j * ldw;
        pv[j] = p[i];
        mv[j] = am[i];
        vv[j] = av[i];
      }
    }
    // K in chunks of 32 rows, the operands of eight chunks in flight
    f32x4 acc = (f32x4)0.0f;
    for (int c = 0; c < B; c += 256) {
      bf16x8 af[8], bf[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (c + 32 * j < B) {
          af[j] = *(const bf16x8*)(ar + c + 32 * j);
          bf[j] = *(const bf16x8*)(br + c + 32 * j);
        }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (c + 32 * j < B) acc = mfma_bf16(af[j], bf[j], acc);
    }
    if (k >= cols) return;
    u16x4 h;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = i0 + (int64_t)j * ldw;
      if (ADAM) {
        adam_element(pv[j], acc[j], mv[j], vv[j], ad);
        p[i] = pv[j];
        am[i] = mv[j];
        av[i] = vv[j];
        h[j] = to_bf16(pv[j]);
        wc[(int64_t)(16 * nt + 4 * q + j) * ldc + k] = h[j];
      } else {
        grad[i] = acc[j];
      }
    }
    if (ADAM && wt) *(u16x4*)(wt + (int64_t)k * ldt + 16 * nt + 4 * q) = h;
    return;
  }
  blk -= kTileBlocks;
  if (blk < kBiasBlocks) {
    __shared__ float part[16][16];
    const float* a = blk < 16 ? w.dz1 : blk < 32 ? w.dz2 : w.dy;
    const int N = blk < 32 ? kHid : kOut;
    const int c0 = (blk < 16 ? blk : blk < 32 ? blk - 16 : blk - 32) * 16;
    const int64_t off = (blk < 16 ? kOffB1 : blk < 32 ? kOffB2 : kOffB3) + c0;
    const int col = threadIdx.x & 15, res = threadIdx.x >> 4;
    const float* col0 = a + (int64_t)res * N + c0 + col;
    float s = 0.0f;
    for (int m = 0; m < B; m += 256) {
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = m + 16 * j < B ? col0[(int64_t)(m + 16 * j) * N] : 0.0f;
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (m + 16 * j < B) s += v[j];
    }
    part[res][col] = s;
    __syncthreads();
    if (threadIdx.x < 16) {
      float g[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) g[j] = (part[j][col] + part[j + 4][col]) + (part[j + 8][col] + part[j + 12][col]);
      const float sum = (g[0] + g[1]) + (g[2] + g[3]);
      const int64_t i = off + col;
      if (ADAM) adam_element(p[i], sum, am[i], av[i], ad);
      else grad[i] = sum;
    }
    return;
  }
  if (!loss) return;
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < B / kRows; i += 256) s += w.lossp[i];
  s = wave_sum_stride<1>(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) *loss = (float)(((red[0] + red[1]) + (red[2] + red[3])) / (double)(B * kOut));
}

// ------------------------------------------------------------ host side ---

static size_t r256(size_t b) { return (b + 255) & ~(size_t)255; }

static size_t mlp_layout(int B, MlpWork* w, char* base) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? base + off : nullptr;
    off += r256(bytes);
    return p;
  };
  const size_t bh = sizeof(bf16_t), f = sizeof(float);
  MlpWork t;
  t.xt = (bf16_t*)take((size_t)B * kIn * bh);
  t.h1t = (bf16_t*)take((size_t)B * kHid * bh);
  t.h2t = (bf16_t*)take((size_t)B * kHid * bh);
  t.dyt = (bf16_t*)take((size_t)B * kOut * bh);
  t.dz2t = (bf16_t*)take((size_t)B * kHid * bh);
  t.dz1t = (bf16_t*)take((size_t)B * kHid * bh);
  t.w1 = (bf16_t*)take((size_t)kHid * kInPad * bh);
  t.w2 = (bf16_t*)take((size_t)kHid * kHid * bh);
  t.w2t = (bf16_t*)take((size_t)kHid * kHid * bh);
  t.w3 = (bf16_t*)take((size_t)kOut * kHid * bh);
  t.w3t = (bf16_t*)take((size_t)kOut * kHid * bh);
  t.dy = (float*)take((size_t)B * kOut * f);
  t.dz2 = (float*)take((size_t)B * kHid * f);
  t.dz1 = (float*)take((size_t)B * kHid * f);
  t.lossp = (double*)take((size_t)B / kRows * sizeof(double));
  if (w) *w = t;
  return off;
}

static void weights_bf16(const float* p, const MlpWork& w, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_weights, dim3((kHid * kHid + 255) / 256), dim3(256), 0, st, p, w.w1, w.w2, w.w2t, w.w3,
                     w.w3t);
}

// Forward and backward pass of the batch, then its gradients (to grad) or
// the Adam step on them.
static void rows_pass(const float* p, int B, const float* xi, const float* tgt, const int32_t* idx, const MlpWork& w,
                      float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_rows<true>, dim3(B / kRows), dim3(1024), 0, st, B, p, xi, tgt, idx, w, out);
}

// out = the network's outputs, through the scratch rows `through` [B][kOut] when
// out shares memory with what the workgroups still read.
static ens_status forward_pass(const float* p, int B, const float* xi, const MlpWork& w, float* out, float* through,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_rows<false>, dim3(B / kRows), dim3(1024), 0, st, B, p, xi, (const float*)nullptr,
                     (const int32_t*)nullptr, w, through ? through : out);
  if (through)
    ENS_HIP_TRY(hipMemcpyAsync(out, through, (size_t)B * kOut * sizeof(float), hipMemcpyDeviceToDevice, st));
  return ENS_OK;
}

// Whether `count` floats at a share memory with the outputs of B rows.
static bool shares(const float* out, int B, const float* a, int64_t count) {
  return a < out + (int64_t)B * kOut && out < a + count;
}

static bool batch_ok(int B) { return B >= 32 && B <= 65536 && B % 32 == 0; }

}  // namespace ens

using namespace ens;

extern "C" {

int64_t ens_mlp_param_count(void) { return kParams; }

ens_status ens_mlp_workspace_bytes(int32_t batch, size_t* bytes) {
  ENS_ARG_CHECK(bytes && batch_ok(batch), "batch must be a multiple of 32 in [32, 65536]");
  *bytes = mlp_layout(batch, nullptr, nullptr);
  return ENS_OK;
}

ens_status ens_mlp_forward(const float* params, int32_t batch, const float* xi, float* out, void* workspace,
                           size_t ws_bytes, hipStream_t stream) {
  ENS_ARG_CHECK(params && xi && out && workspace, "null pointer");
  ENS_ARG_CHECK(batch_ok(batch), "batch must be a multiple of 32 in [32, 65536]");
  ENS_ARG_CHECK(((uintptr_t)workspace & 255u) == 0, "workspace must be 256-byte aligned");
  if (ws_bytes < mlp_layout(batch, nullptr, nullptr)) {
    set_error("MLP workspace too small");
    return ENS_E_NOMEM;
  }
  MlpWork w;
  mlp_layout(batch, &w, (char*)workspace);
  weights_bf16(params, w, stream);
  const bool in_place = shares(out, batch, xi, (int64_t)batch * kIn) || shares(out, batch, params, kParams);
  const ens_status rc = forward_pass(params, batch, xi, w, out, in_place ? w.dy : nullptr, stream);
  if (rc != ENS_OK) return rc;
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_mlp_grad(const float* params, int32_t batch, const float* xi, const float* target, float* out,
                        float* grad, float* loss, void* workspace, size_t ws_bytes, hipStream_t stream) {
  ENS_ARG_CHECK(params && xi && target && grad && workspace, "null pointer");
  ENS_ARG_CHECK(batch_ok(batch), "batch must be a multiple of 32 in [32, 65536]");
  ENS_ARG_CHECK(((uintptr_t)workspace & 255u) == 0, "workspace must be 256-byte aligned");
  if (ws_bytes < mlp_layout(batch, nullptr, nullptr)) {
    set_error("MLP workspace too small");
    return ENS_E_NOMEM;
  }
  MlpWork w;
  mlp_layout(batch, &w, (char*)workspace);
  weights_bf16(params, w, stream);
  // (out in the place of target itself: each lane reads a target before it
  // writes there)
  const bool in_place = out && (shares(out, batch, xi, (int64_t)batch * kIn) || shares(out, batch, params, kParams) ||
                                (out != target && shares(out, batch, target, (int64_t)batch * kOut)));
  rows_pass(params, batch, xi, target, nullptr, w, in_place ? nullptr : out, stream);
  hipLaunchKernelGGL(k_mlp_update<false>, dim3(kUpdateBlocks), dim3(256), 0, stream, batch, w, (float*)nullptr,
                     (float*)nullptr, (float*)nullptr, AdamStep{}, grad, loss);
  if (in_place) {  // a forward pass of its own; the update is done with dz1
    const ens_status rc = forward_pass(params, batch, xi, w, out, w.dz1, stream);
    if (rc != ENS_OK) return rc;
  }
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

ens_status ens_mlp_train(float* params, float* adam_m, float* adam_v, int32_t step0, const float* xi,
                         const float* target, int32_t count, int32_t batch, int32_t steps, const int32_t* batch_idx,
                         float lr, float* loss, void* workspace, size_t ws_bytes, hipStream_t stream) {
  ENS_ARG_CHECK(params && adam_m && adam_v && xi && target && batch_idx && workspace, "null pointer");
  ENS_ARG_CHECK(batch_ok(batch) && count >= 1 && steps >= 0 && step0 >= 0, "bad sizes");
  ENS_ARG_CHECK(((uintptr_t)workspace & 255u) == 0, "workspace must be 256-byte aligned");
  ENS_ARG_CHECK(lr > 0.0f, "learning rate must be positive");
  if (ws_bytes < mlp_layout(batch, nullptr, nullptr)) {
    set_error("MLP workspace too small");
    return ENS_E_NOMEM;
  }
  MlpWork w;
  mlp_layout(batch, &w, (char*)workspace);
  weights_bf16(params, w, stream);
  AdamPowers pw;
  pw.advance(step0);
  for (int s = 0; s < steps; ++s) {
    pw.advance(1);
    rows_pass(params, batch, xi, target, batch_idx + (int64_t)s * batch, w, nullptr, stream);
    hipLaunchKernelGGL(k_mlp_update<true>, dim3(kUpdateBlocks), dim3(256), 0, stream, batch, w, params, adam_m, adam_v,
                       pw.step(lr), (float*)nullptr, loss ? loss + s : nullptr);
    ENS_LAUNCH_CHECK();
  }
  return ENS_OK;
}

ens_status ens_mlp_adam(float* params, const float* grad, float* adam_m, float* adam_v, int64_t count, int32_t step,
                        float lr, hipStream_t stream) {
  ENS_ARG_CHECK(params && grad && adam_m && adam_v, "null pointer");
  ENS_ARG_CHECK(count >= 0 && step >= 1, "count must be >= 0 and step >= 1");
  ENS_ARG_CHECK(lr > 0.0f, "learning rate must be positive");
  ENS_ARG_CHECK(count <= INT32_MAX, "count must fit in int32");
  if (count == 0) return ENS_OK;
  AdamPowers pw;
  pw.advance(step);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, count, params, grad, adam_m,
                     adam_v, pw.step(lr));
  ENS_LAUNCH_CHECK();
  return ENS_OK;
}

}  // extern "C"
