// mlp.hip -- the change predictor: a 12 -> 64 -> 64 -> 1 perceptron with ReLU
// hidden layers and a sigmoid output, stored as fp32 master parameters with
// bfloat16 copies for inference.  (A project addition, not in the paper.)
//
// Parameter order (flat, fp32): W1 [12][64], b1 [64], W2 [64][64], b2 [64],
// W3 [64], b3 [1]; W[k][j] multiplies input k into unit j.
//
//   k_mlp_grad    forward + backward of a minibatch in fp32 on bf16-rounded
//                 weights and inputs, on v_mfma_f32_16x16x4_f32; each
//                 workgroup writes the gradient of its 64 samples
//   k_mlp_reduce  sums the workgroups' gradients (and losses) in fp64 and,
//                 in training, takes the Adam step on the sum
//   k_adam        one Adam step (Kingma & Ba 2015) with bias correction
//   k_mlp_pack    fp32 masters -> bf16 MFMA operand tiles
//   mlp_logit16   inference of 16 samples by one wave with
//                 v_mfma_f32_16x16x16_bf16: every layer is computed
//                 transposed (weights as the A operand, samples as the 16
//                 columns), so a layer's output tile, after bias, ReLU and
//                 bf16 rounding, is the next layer's B operand unchanged
#include <cmath>

#include "lpa_mlp.h"

namespace lpa {

namespace {

constexpr int kIn = 12, kH = 64;
constexpr int oW1 = 0, ob1 = oW1 + kIn * kH, oW2 = ob1 + kH, ob2 = oW2 + kH * kH,
              oW3 = ob2 + kH, ob3 = oW3 + kH;
static_assert(ob3 + 1 == kMlpParams, "parameter count");

constexpr int kGradTiles = 2;     // of 16 samples per wave
constexpr int kGradThreads = 512;
constexpr int kGradStride = 80;   // floats between two samples' units in LDS
constexpr int kH2Stride = 68;     // the same for reads of one sample per lane
static_assert(kGradSamples == 2 * 16 * kGradTiles, "a wave half per half of the samples");

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

}  // namespace

// ---- training -------------------------------------------------------------------
// Forward and backward pass of the samples s0, s0 + 1, ... (idx: through this
// list), kGradSamples = 64 per workgroup and round; the workgroup's gradient
// goes to part + blockIdx.x * kMlpPartStride, the loss of each 64 samples to
// loss[].
//
// Training amplifies a gradient's last bit (the weights are rounded to bf16 at
// every step: one ulp of a master weight near a rounding boundary moves the
// next gradient by 2^-9 of that weight), so the order of every sum is part of
// what the kernel computes: per output one chain of fused multiply-adds, over
// the inputs in the forward products, over the units in da1, and in every
// weight and bias gradient over the 64 samples in their order.
// v_mfma_f32_16x16x4_f32 is such a chain over its four k (fp32 operands and
// sums), so all products run as its 16 x 16 tiles, and a sum of plain values
// has ones as its other operand.
//
// The eight waves are four unit groups (units 16 u .. 16 u + 15 of every layer)
// times two halves of the samples.  In the products over inputs and units the
// units are rows and the samples columns, so that lane (j, k) = (lane % 16,
// lane / 16) holds units 16 u + 4 k + r, r = 0 .. 3, of sample j of a tile.
// In the gradients the samples are the inner dimension: the halves then split
// the rows of W2's, and at the end one half takes W1 and b1 (the row of ones
// that W1's 12 inputs leave free), the other W3 and b2.  Samples lie 80 floats
// apart in LDS, which spreads the four sample rows of a read over different
// banks.  A wave's weights and gradient tiles stay in registers over the rounds.
//
// It is bound by latency at a minibatch's size: 4,096 samples are one round of
// 64 workgroups, 128 to 144 products of 32 cycles per wave between six
// barriers.  Measured there: 37 us with scalar LDS loops and 5,057 atomic adds
// per workgroup, 20 us with this kernel and 4 us for k_mlp_reduce (17 us with
// 32 samples and four waves a workgroup on twice the CUs, which sums in another
// order); 10^6 samples 1.3 -> 0.55 ms.  The two tiles' chains taken in turn
// product by product: 20 us as well.
__global__ __launch_bounds__(kGradThreads) void k_mlp_grad(
    const float* __restrict__ p, const float* __restrict__ X, const float* __restrict__ y,
    const int32_t* __restrict__ idx, int64_t B, float inv_total, float pos_weight,
    float* __restrict__ part, float* __restrict__ loss) {
  __shared__ __align__(16) float h1s[kGradSamples * kGradStride];   // later da1
  __shared__ __align__(16) float da2s[kGradSamples * kGradStride];
  __shared__ __align__(16) float h2s[kGradSamples * kH2Stride];
  __shared__ __align__(16) float w3s[kH];
  __shared__ float xs[kGradSamples][kIn + 1];
  const int tid = threadIdx.x, lane = tid & 63, u = (tid >> 6) & 3, half = tid >> 8;
  const int j = lane & 15, k = lane >> 4;
  const int c0 = 16 * u + j;                       // the lane's column in a gradient tile
  const int sm0 = 16 * kGradTiles * half + j;      // the lane's sample in the first tile
  // a round's features and targets, loaded a round ahead: the thread's share of
  // xs, and in every wave the target of sample lane
  constexpr int kX = (kGradSamples * kIn + kGradThreads - 1) / kGradThreads;
  float xv[kX], tn = 0.0f;
  auto fetch = [&](int64_t s0) {
    const int64_t last = B - 1;
    int64_t row[kX], ty = 0;
#pragma unroll
    for (int q = 0; q < kX; ++q) {
      const int i = tid + q * kGradThreads;
      const int64_t s = s0 + i / kIn;
      row[q] = s < B ? s : last;
      if (idx) row[q] = idx[row[q]];
    }
    ty = s0 + lane < B ? s0 + lane : last;
    if (idx) ty = idx[ty];
#pragma unroll
    for (int q = 0; q < kX; ++q) xv[q] = X[row[q] * kIn + (tid + q * kGradThreads) % kIn];
    tn = y[ty];
  };
  fetch((int64_t)blockIdx.x * kGradSamples);
  // the wave's weights: w1a[q] = W1[4 q + k][c0]; w2f[q] = W2[4 q + k][c0];
  // w2b[q] = W2[c0][4 q + k]
  float w1a[3], w2f[16], w2b[16];
  v4f b1v, b2v, w3v;
#pragma unroll
  for (int q = 0; q < 3; ++q) w1a[q] = bf16_round(p[oW1 + (4 * q + k) * kH + c0]);
#pragma unroll
  for (int q = 0; q < 16; ++q) w2f[q] = bf16_round(p[oW2 + (4 * q + k) * kH + c0]);
#pragma unroll
  for (int q = 0; q < 16; ++q) w2b[q] = bf16_round(p[oW2 + c0 * kH + 4 * q + k]);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    b1v[r] = p[ob1 + 16 * u + 4 * k + r];
    b2v[r] = p[ob2 + 16 * u + 4 * k + r];
    w3v[r] = bf16_round(p[oW3 + 16 * u + 4 * k + r]);
  }
  if (tid < kH) w3s[tid] = bf16_round(p[oW3 + tid]);
  const float b3 = p[ob3];
  const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  v4f g2[2] = {zero, zero};        // W2: rows 32 half + 16 m + 4 k + r, column c0
  v4f ga = zero, gb = zero;        // half 0: W1 and b1, b3; half 1: W3, b2
  for (int64_t s0 = (int64_t)blockIdx.x * kGradSamples; s0 < B;
       s0 += (int64_t)gridDim.x * kGradSamples) {
    const int ns = (int)((B - s0) < kGradSamples ? (B - s0) : kGradSamples);
#pragma unroll
    for (int q = 0; q < kX; ++q) {
      const int i = tid + q * kGradThreads;
      if (i < kGradSamples * kIn) xs[i / kIn][i % kIn] = i / kIn < ns ? bf16_round(xv[q]) : 0.0f;
    }
    const float t = tn;  // target of sample lane
    const int64_t next = s0 + (int64_t)gridDim.x * kGradSamples;
    if (next < B) fetch(next);
    __syncthreads();
    // layer 1
    v4f h1[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      const int sm = sm0 + 16 * a;
      v4f acc = b1v;
#pragma unroll
      for (int q = 0; q < 3; ++q) acc = mfma4(w1a[q], xs[sm][4 * q + k], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) h1[a][r] = fmaxf(acc[r], 0.0f);
      *reinterpret_cast<v4f*>(&h1s[sm * kGradStride + 16 * u + 4 * k]) = h1[a];
    }
    __syncthreads();
    // layer 2
    v4f h2[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      const int sm = sm0 + 16 * a;
      v4f acc = b2v;
#pragma unroll
      for (int q = 0; q < 16; ++q) acc = mfma4(w2f[q], h1s[sm * kGradStride + 4 * q + k], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[a][r] = fmaxf(acc[r], 0.0f);
      *reinterpret_cast<v4f*>(&h2s[sm * kH2Stride + 16 * u + 4 * k]) = h2[a];
    }
    __syncthreads();
    // logit and d loss / d logit of sample lane, in every wave
    float dz = 0.0f, my_loss = 0.0f;
    if (lane < ns) {
      float z = b3;
#pragma unroll
      for (int i = 0; i < kH; i += 4) {
        const v4f h = *reinterpret_cast<const v4f*>(&h2s[lane * kH2Stride + i]);
        const v4f c = *reinterpret_cast<const v4f*>(&w3s[i]);
#pragma unroll
        for (int r = 0; r < 4; ++r) z += h[r] * c[r];
      }
      const float sg = 1.0f / (1.0f + __expf(-z));
      // d/dz of -[pw t log s + (1 - t) log(1 - s)]
      dz = (pos_weight * t * (sg - 1.0f) + (1.0f - t) * sg) * inv_total;
      if (tid < 64) {
        // log sigmoid(z) and log(1 - sigmoid(z)), stable
        const float ls = -(fmaxf(-z, 0.0f) + log1pf(__expf(-fabsf(z))));
        const float l1s = -(fmaxf(z, 0.0f) + log1pf(__expf(-fabsf(z))));
        my_loss = -(pos_weight * t * ls + (1.0f - t) * l1s);
      }
    }
    if (tid < 64) {
      for (int ofs = 32; ofs > 0; ofs >>= 1) my_loss += __shfl_xor(my_loss, ofs);
      if (lane == 0) loss[s0 / kGradSamples] = my_loss;
    }
    // da2 = dz W3 [h2 > 0]
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      const int sm = sm0 + 16 * a;
      const float d = __shfl(dz, sm);
      v4f da2;
#pragma unroll
      for (int r = 0; r < 4; ++r) da2[r] = h2[a][r] > 0.0f ? d * w3v[r] : 0.0f;
      *reinterpret_cast<v4f*>(&da2s[sm * kGradStride + 16 * u + 4 * k]) = da2;
    }
    __syncthreads();
    // W2 gradient, the wave's columns and half of the rows: sum over samples of
    // h1[s][.] da2[s][.]
#pragma unroll
    for (int q = 0; q < kGradSamples / 4; ++q) {
      const float b = da2s[(4 * q + k) * kGradStride + c0];
#pragma unroll
      for (int m = 0; m < 2; ++m)
        g2[m] = mfma4(h1s[(4 * q + k) * kGradStride + 32 * half + 16 * m + j], b, g2[m]);
    }
    // da1 = da2 W2^T [h1 > 0], the wave's units and samples
    v4f da1[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      v4f acc = zero;
#pragma unroll
      for (int q = 0; q < 16; ++q)
        acc = mfma4(w2b[q], da2s[(sm0 + 16 * a) * kGradStride + 4 * q + k], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) da1[a][r] = h1[a][r] > 0.0f ? acc[r] : 0.0f;
    }
    __syncthreads();  // every wave has read h1s
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a)
      *reinterpret_cast<v4f*>(&h1s[(sm0 + 16 * a) * kGradStride + 16 * u + 4 * k]) = da1[a];
    __syncthreads();
    if (half == 0) {
      // rows 0 .. 11: W1 gradient, the wave's columns; row 12: b1's; and b3's
#pragma unroll
      for (int q = 0; q < kGradSamples / 4; ++q) {
        const float a = j < kIn ? xs[4 * q + k][j] : (j == kIn ? 1.0f : 0.0f);
        ga = mfma4(a, h1s[(4 * q + k) * kGradStride + c0], ga);
        if (u == 0) gb = mfma4(1.0f, __shfl(dz, 4 * q + k), gb);
      }
    } else {
      // W3 and b2 gradients of the wave's units, the same in every column
#pragma unroll
      for (int q = 0; q < kGradSamples / 4; ++q) {
        ga = mfma4(h2s[(4 * q + k) * kH2Stride + c0], __shfl(dz, 4 * q + k), ga);
        gb = mfma4(da2s[(4 * q + k) * kGradStride + c0], 1.0f, gb);
      }
    }
    __syncthreads();  // the LDS arrays are rewritten by the next round
  }
  float* out = part + (size_t)blockIdx.x * kMlpPartStride;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * k + r;
#pragma unroll
    for (int m = 0; m < 2; ++m) out[oW2 + (32 * half + 16 * m + row) * kH + c0] = g2[m][r];
    if (half == 0) {
      if (row < kIn) out[oW1 + row * kH + c0] = ga[r];
      if (row == kIn) out[ob1 + c0] = ga[r];
    } else if (j == 0) {
      out[oW3 + 16 * u + row] = ga[r];
      out[ob2 + 16 * u + row] = gb[r];
    }
  }
  if (tid == 0) out[ob3] = gb[0];
}

// The products that are rounded and those that are fused are written out: the
// compiler's choice differs from kernel to kernel.
__device__ __forceinline__ void adam_update(float* p, float* m, float* v, int i, float gi,
                                            const AdamStep& a) {
  const float mi = fmaf(a.omb1, gi, a.beta1 * m[i]);
  const float vi = fmaf(gi, a.omb2 * gi, a.beta2 * v[i]);
  m[i] = mi;
  v[i] = vi;
  p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// The gradient from the parts of np workgroups, summed in fp64: 64 parameters
// per workgroup, the parts split over its four waves.  STEP: also the Adam
// step.  The first workgroup sums the nl losses in fp64: to *loss, or (add) on
// top of it.  Every sum is in a fixed order.
template <bool STEP>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ part,
                                                    const float* __restrict__ ploss, int np,
                                                    int64_t nl, float* g, double* loss, int add,
                                                    float* p, float* m, float* v, AdamStep a) {
  __shared__ double sums[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (i < kMlpParams) {
    int q = w;
    for (; q + 28 < np; q += 32) {  // eight loads in flight
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = part[(size_t)(q + 4 * u) * kMlpPartStride + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += (double)x[u];
    }
    for (; q < np; q += 4) s += (double)part[(size_t)q * kMlpPartStride + i];
  }
  sums[w][lane] = s;
  __syncthreads();
  if (w == 0 && i < kMlpParams) {
    const float gi = (float)(sums[0][lane] + sums[1][lane] + sums[2][lane] + sums[3][lane]);
    g[i] = gi;
    if constexpr (STEP) adam_update(p, m, v, i, gi, a);
  }
  if (blockIdx.x != 0) return;
  double t = 0.0;
  for (int64_t q = threadIdx.x; q < nl; q += 256) t += (double)ploss[q];
  for (int ofs = 32; ofs > 0; ofs >>= 1) t += __shfl_xor(t, ofs);
  __syncthreads();
  if (lane == 0) sums[w][0] = t;
  __syncthreads();
  if (threadIdx.x == 0)
    *loss = (add ? *loss : 0.0) + (sums[0][0] + sums[1][0] + sums[2][0] + sums[3][0]);
}

__global__ void k_adam(float* p, const float* g, float* m, float* v, int n, AdamStep a) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    adam_update(p, m, v, i, g[i], a);
}

// ---- inference ----------------------------------------------------------------------
// Operand tiles, one 8-byte group of 4 bf16 per lane and tile:
//   w1t[m][lane]     = W1[4 (lane/16) + j][16 m + lane%16], j = 0..3, zero for
//                      input rows >= 12                       (m = 0..3)
//   w2t[mo][kb][lane] = W2[16 kb + 4 (lane/16) + j][16 mo + lane%16]
__global__ void k_mlp_pack(const float* p, MlpTiles* t) {
  for (int i = threadIdx.x; i < 4 * 64; i += blockDim.x) {
    const int m = i / 64, lane = i % 64;
    for (int j = 0; j < 4; ++j) {
      const int k = 4 * (lane / 16) + j, col = 16 * m + lane % 16;
      t->w1t[m][lane][j] = k < kIn ? bf16_bits(p[oW1 + k * kH + col]) : (uint16_t)0;
    }
  }
  for (int i = threadIdx.x; i < 16 * 64; i += blockDim.x) {
    const int mo = i / 256, kb = (i / 64) % 4, lane = i % 64;
    for (int j = 0; j < 4; ++j) {
      const int k = 16 * kb + 4 * (lane / 16) + j, col = 16 * mo + lane % 16;
      t->w2t[mo][kb][lane][j] = bf16_bits(p[oW2 + k * kH + col]);
    }
  }
  for (int i = threadIdx.x; i < kH; i += blockDim.x) {
    t->b1[i] = p[ob1 + i];
    t->b2[i] = p[ob2 + i];
    t->w3[i] = bf16_round(p[oW3 + i]);
  }
  if (threadIdx.x == 0) t->b3 = p[ob3];
}

// One wave takes 16 samples a step; the next step's features are loaded while
// the network runs on the current ones.  X4: X is 16-byte aligned, so that a
// lane's four features are one load.
template <bool X4>
__global__ __launch_bounds__(256) void k_mlp_infer(const MlpTiles* t, const float* X, int64_t B,
                                                   float* out) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  // group 3 holds the padding of the 12 features: its loads repeat group 2's
  const int col = g < 3 ? 4 * g : 8;
  float f[4];
  auto load = [&](int64_t s0) {
    const int64_t s = s0 + (lane & 15);
    const float* x = X + (s < B ? s : B - 1) * kIn + col;
    if constexpr (X4) {
      const v4f v = *reinterpret_cast<const v4f*>(x);
#pragma unroll
      for (int q = 0; q < 4; ++q) f[q] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) f[q] = x[q];
    }
  };
  MlpLane r;
  mlp_load(*t, r);
  if (wave * 16 < B) load(wave * 16);
  for (int64_t s0 = wave * 16; s0 < B; s0 += nw * 16) {
    float c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = g < 3 ? f[q] : 0.0f;
    load(s0 + nw * 16);
    const float z = mlp_logit16(r, c);
    const int64_t s = s0 + lane;
    if (lane < 16 && s < B) out[s] = 1.0f / (1.0f + __expf(-z));
  }
}

int64_t mlp_grad_losses(int64_t B) { return (B + kGradSamples - 1) / kGradSamples; }

int mlp_grad_parts(int64_t B) {
  const int64_t g = mlp_grad_losses(B);
  return (int)(g < kMlpMaxParts ? g : kMlpMaxParts);
}

static AdamStep adam_step(int t, float lr) {
  // 1 - beta and the bias corrections, each rounded once from fp64 (1 - 0.999f
  // in fp32 would be off by 1e-5 relative)
  const double beta1 = 0.9, beta2 = 0.999;
  AdamStep a;
  a.lr = lr;
  a.beta1 = (float)beta1;
  a.omb1 = (float)(1.0 - beta1);
  a.beta2 = (float)beta2;
  a.omb2 = (float)(1.0 - beta2);
  a.eps = 1e-8f;
  a.c1 = (float)(1.0 - std::pow(beta1, (double)t));
  a.c2 = (float)(1.0 - std::pow(beta2, (double)t));
  return a;
}

hipError_t launch_mlp_grad(const float* p, const float* X, const float* y, const int32_t* idx,
                           int64_t B, float pos_weight, float* part, float* ploss, hipStream_t s) {
  if (B <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)mlp_grad_parts(B)), dim3(kGradThreads), 0, s, p,
                     X, y, idx, B, 1.0f / (float)B, pos_weight, part, ploss);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const float* part, const float* ploss, int64_t B, float* g,
                             double* loss, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kMlpParams + 63) / 64), dim3(256), 0, s, part,
                     ploss, mlp_grad_parts(B), mlp_grad_losses(B), g, loss, 0, nullptr, nullptr,
                     nullptr, AdamStep{});
  return hipGetLastError();
}

hipError_t launch_mlp_reduce_step(const float* part, const float* ploss, int64_t B, float* g,
                                  double* loss, bool add, float* p, float* m, float* v, int t,
                                  float lr, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kMlpParams + 63) / 64), dim3(256), 0, s, part,
                     ploss, mlp_grad_parts(B), mlp_grad_losses(B), g, loss, add ? 1 : 0, p, m, v,
                     adam_step(t, lr));
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int t, float lr,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, p, g, m, v,
                     kMlpParams, adam_step(t, lr));
  return hipGetLastError();
}

hipError_t launch_mlp_pack(const float* p, MlpTiles* t, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_pack, dim3(1), dim3(256), 0, s, p, t);
  return hipGetLastError();
}

// Up to four workgroups per CU (their weights, 10 KB a wave, are loaded once).
hipError_t launch_mlp_infer(const MlpTiles* t, const float* X, int64_t B, float* out,
                            hipStream_t s) {
  if (B <= 0) return hipSuccess;
  int64_t g = (B + 63) / 64;
  if (g > 1024) g = 1024;
  if (reinterpret_cast<uintptr_t>(X) % 16 == 0)
    hipLaunchKernelGGL(k_mlp_infer<true>, dim3((unsigned)g), dim3(256), 0, s, t, X, B, out);
  else
    hipLaunchKernelGGL(k_mlp_infer<false>, dim3((unsigned)g), dim3(256), 0, s, t, X, B, out);
  return hipGetLastError();
}

}  // namespace lpa
