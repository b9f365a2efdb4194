// mlp.hip -- the change predictor: a 12 -> 64 -> 64 -> 1 perceptron with ReLU
// hidden layers and a sigmoid output, stored as fp32 master parameters with
// bfloat16 copies for inference.  (A project addition, not in the paper.)
//
// Parameter order (flat, fp32): W1 [12][64], b1 [64], W2 [64][64], b2 [64],
// W3 [64], b3 [1]; W[k][j] multiplies input k into unit j.
//
//   k_mlp_grad    forward + backward of a minibatch in fp32 on bf16-rounded
//                 weights and inputs, on v_mfma_f32_16x16x4_f32; each
//                 workgroup writes the gradient of its samples
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

constexpr int kGradSamples = 32;  // samples per workgroup and round
constexpr int kGradTiles = kGradSamples / 16;
constexpr int kGradThreads = 256;
constexpr int kGradStride = 80;   // floats between two samples' units in LDS
constexpr int kH2Stride = 68;     // the same for reads of one sample per lane

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Sum over the 16 lanes of a DPP row, in every lane of it.
__device__ __forceinline__ float dpp_row_sum(float x) {
  x += __shfl_xor(x, 1);
  x += __shfl_xor(x, 2);
  x += __shfl_xor(x, 4);
  x += __shfl_xor(x, 8);
  return x;
}

}  // namespace

// ---- training -------------------------------------------------------------------
// Forward and backward pass of the samples s0, s0 + 1, ... (idx: through this
// list), kGradSamples per workgroup and round; the workgroup's gradient goes
// to part + blockIdx.x * kMlpPartStride, each sample's loss to loss[], and
// *total is cleared for the reduction unless add.
//
// The four waves share the samples and split the hidden units: wave w has
// units 16 w .. 16 w + 15 of every layer.  All products run as 16 x 16 tiles
// of v_mfma_f32_16x16x4_f32 (fp32 operands and sums, as before on the vector
// units) with the units as rows and the samples as columns, so that lane
// (j, k) = (lane % 16, lane / 16) holds units 16 w + 4 k + r, r = 0 .. 3, of
// sample j.  The forward sums run over the inputs in their order, one fused
// multiply-add after the other, so that a sample's logit and loss do not
// depend on how the samples are split; the backward product over the units
// takes them in the order 16 m + 4 k + r that one 16-byte read per four
// products gives.  The weight gradients sum over samples: there the samples
// are the inner dimension, and both operands are read from LDS with a stride
// of 80 floats, which spreads the four sample rows of a read over different
// banks.  A wave's weights (the W2 columns and rows of its units) and
// gradient tiles stay in registers over the rounds.
//
// It is bound by latency at a minibatch's size (4,096 samples are one round
// of 128 workgroups: 110 products of 32 cycles per wave between five
// barriers).  Measured there: 37 us with scalar LDS loops and 5,057 atomic
// adds per workgroup, 16 us with this kernel and 4 us for k_mlp_reduce; 10^6
// samples 1.3 -> 0.4 ms.
__global__ __launch_bounds__(kGradThreads) void k_mlp_grad(
    const float* __restrict__ p, const float* __restrict__ X, const float* __restrict__ y,
    const int32_t* __restrict__ idx, int64_t B, float inv_total, float pos_weight,
    float* __restrict__ part, float* __restrict__ loss, double* total, int add) {
  __shared__ __align__(16) float h1s[kGradSamples * kGradStride];   // later da1
  __shared__ __align__(16) float da2s[kGradSamples * kGradStride];
  __shared__ __align__(16) float h2s[kGradSamples * kH2Stride];
  __shared__ __align__(16) float w3s[kH];
  __shared__ float xs[kGradSamples][kIn + 1];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j = lane & 15, k = lane >> 4;
  // a round's features and targets, loaded a round ahead: the thread's share of
  // xs, and in lanes 0 .. 31 of every wave the sample's target
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
    ty = s0 + (lane & 31) < B ? s0 + (lane & 31) : last;
    if (idx) ty = idx[ty];
#pragma unroll
    for (int q = 0; q < kX; ++q) xv[q] = X[row[q] * kIn + (tid + q * kGradThreads) % kIn];
    tn = y[ty];
  };
  fetch((int64_t)blockIdx.x * kGradSamples);
  // the wave's weights: w1a[q] = W1[4 q + k][16 w + j]; w2f[q] = W2[4 q + k][16 w
  // + j]; w2b[m][r] = W2[16 w + j][16 m + 4 k + r]
  float w1a[3], w2f[16], w2b[4][4];
  v4f b1v, b2v, w3v;
#pragma unroll
  for (int q = 0; q < 3; ++q) w1a[q] = bf16_round(p[oW1 + (4 * q + k) * kH + 16 * w + j]);
#pragma unroll
  for (int q = 0; q < 16; ++q) w2f[q] = bf16_round(p[oW2 + (4 * q + k) * kH + 16 * w + j]);
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      w2b[m][r] = bf16_round(p[oW2 + (16 * w + j) * kH + 16 * m + 4 * k + r]);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    b1v[r] = p[ob1 + 16 * w + 4 * k + r];
    b2v[r] = p[ob2 + 16 * w + 4 * k + r];
    w3v[r] = bf16_round(p[oW3 + 16 * w + 4 * k + r]);
  }
  if (tid < kH) w3s[tid] = bf16_round(p[oW3 + tid]);
  if (blockIdx.x == 0 && tid == 0 && !add) *total = 0.0;
  const float b3 = p[ob3];
  const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  v4f g2[4] = {zero, zero, zero, zero}, g1 = zero;  // rows 16 m + 4 k + r, column 16 w + j
  v4f gb1 = zero, gb2 = zero, g3 = zero;            // units 16 w + 4 k + r, of column j
  float gb3 = 0.0f;
  for (int64_t s0 = (int64_t)blockIdx.x * kGradSamples; s0 < B;
       s0 += (int64_t)gridDim.x * kGradSamples) {
    const int ns = (int)((B - s0) < kGradSamples ? (B - s0) : kGradSamples);
#pragma unroll
    for (int q = 0; q < kX; ++q) {
      const int i = tid + q * kGradThreads;
      if (i < kGradSamples * kIn) xs[i / kIn][i % kIn] = i / kIn < ns ? bf16_round(xv[q]) : 0.0f;
    }
    const float t = tn;  // target of sample lane (lanes 0 .. 31)
    const int64_t next = s0 + (int64_t)gridDim.x * kGradSamples;
    if (next < B) fetch(next);
    __syncthreads();
    // layer 1
    v4f h1[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      v4f acc = b1v;
#pragma unroll
      for (int q = 0; q < 3; ++q) acc = mfma4(w1a[q], xs[16 * a + j][4 * q + k], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) h1[a][r] = fmaxf(acc[r], 0.0f);
      *reinterpret_cast<v4f*>(&h1s[(16 * a + j) * kGradStride + 16 * w + 4 * k]) = h1[a];
    }
    __syncthreads();
    // layer 2
    v4f h2[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      v4f acc = b2v;
#pragma unroll
      for (int q = 0; q < 16; ++q)
        acc = mfma4(w2f[q], h1s[(16 * a + j) * kGradStride + 4 * q + k], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[a][r] = fmaxf(acc[r], 0.0f);
      *reinterpret_cast<v4f*>(&h2s[(16 * a + j) * kH2Stride + 16 * w + 4 * k]) = h2[a];
    }
    __syncthreads();
    // logit and d loss / d logit of sample lane, in lanes 0 .. 31 of every wave
    float dz = 0.0f;
    if (lane < ns && lane < kGradSamples) {
      float z = b3;
#pragma unroll
      for (int u = 0; u < kH; u += 4) {
        const v4f h = *reinterpret_cast<const v4f*>(&h2s[lane * kH2Stride + u]);
        const v4f c = *reinterpret_cast<const v4f*>(&w3s[u]);
#pragma unroll
        for (int r = 0; r < 4; ++r) z += h[r] * c[r];
      }
      const float sg = 1.0f / (1.0f + __expf(-z));
      // d/dz of -[pw t log s + (1 - t) log(1 - s)]
      dz = (pos_weight * t * (sg - 1.0f) + (1.0f - t) * sg) * inv_total;
      if (w == 0) {
        // log sigmoid(z) and log(1 - sigmoid(z)), stable
        const float ls = -(fmaxf(-z, 0.0f) + log1pf(__expf(-fabsf(z))));
        const float l1s = -(fmaxf(z, 0.0f) + log1pf(__expf(-fabsf(z))));
        loss[s0 + lane] = -(pos_weight * t * ls + (1.0f - t) * l1s);
      }
    }
    gb3 += dz;
    // da2 = dz W3 [h2 > 0]
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      const float d = __shfl(dz, 16 * a + j);
      v4f da2;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        g3[r] += h2[a][r] * d;
        da2[r] = h2[a][r] > 0.0f ? d * w3v[r] : 0.0f;
        gb2[r] += da2[r];
      }
      *reinterpret_cast<v4f*>(&da2s[(16 * a + j) * kGradStride + 16 * w + 4 * k]) = da2;
    }
    __syncthreads();
    // W2 gradient, the wave's columns: sum over samples of h1[s][.] da2[s][.]
#pragma unroll
    for (int q = 0; q < kGradSamples / 4; ++q) {
      const float b = da2s[(4 * q + k) * kGradStride + 16 * w + j];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        g2[m] = mfma4(h1s[(4 * q + k) * kGradStride + 16 * m + j], b, g2[m]);
    }
    // da1 = da2 W2^T [h1 > 0], the wave's units
    v4f da1[kGradTiles];
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a) {
      v4f acc = zero;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const v4f b = *reinterpret_cast<const v4f*>(
            &da2s[(16 * a + j) * kGradStride + 16 * m + 4 * k]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma4(w2b[m][r], b[r], acc);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        da1[a][r] = h1[a][r] > 0.0f ? acc[r] : 0.0f;
        gb1[r] += da1[a][r];
      }
    }
    __syncthreads();  // every wave has read h1s
#pragma unroll
    for (int a = 0; a < kGradTiles; ++a)
      *reinterpret_cast<v4f*>(&h1s[(16 * a + j) * kGradStride + 16 * w + 4 * k]) = da1[a];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // W1 gradient, the wave's columns (written by the wave itself)
#pragma unroll
    for (int q = 0; q < kGradSamples / 4; ++q)
      g1 = mfma4(j < kIn ? xs[4 * q + k][j] : 0.0f,
                 h1s[(4 * q + k) * kGradStride + 16 * w + j], g1);
    __syncthreads();  // xs, h1s and h2s are rewritten by the next round
  }
  float* out = part + (size_t)blockIdx.x * kMlpPartStride;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (4 * k + r < kIn) out[oW1 + (4 * k + r) * kH + 16 * w + j] = g1[r];
#pragma unroll
    for (int m = 0; m < 4; ++m) out[oW2 + (16 * m + 4 * k + r) * kH + 16 * w + j] = g2[m][r];
    const float x1 = dpp_row_sum(gb1[r]), x2 = dpp_row_sum(gb2[r]), x3 = dpp_row_sum(g3[r]);
    if (j == 0) {
      const int u = 16 * w + 4 * k + r;
      out[ob1 + u] = x1;
      out[ob2 + u] = x2;
      out[oW3 + u] = x3;
    }
  }
  if (w == 0) {
    for (int ofs = 32; ofs > 0; ofs >>= 1) gb3 += __shfl_xor(gb3, ofs);
    if (lane == 0) out[ob3] = gb3;
  }
}

__device__ __forceinline__ void adam_update(float* p, float* m, float* v, int i, float gi,
                                            const AdamStep& a) {
  const float mi = a.beta1 * m[i] + a.omb1 * gi;
  const float vi = a.beta2 * v[i] + a.omb2 * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// The gradient from the parts of np workgroups, summed in fp64: 64 parameters
// per workgroup, the parts split over its four waves.  STEP: also the Adam
// step.  The losses of the B samples are added to *loss, in fp32 over each 64
// consecutive samples and in fp64 over those.
template <bool STEP>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ part,
                                                    const float* __restrict__ ploss, int np,
                                                    int64_t B, float* g, double* loss, float* p,
                                                    float* m, float* v, AdamStep a) {
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
  double t = 0.0;
  for (int64_t s0 = ((int64_t)blockIdx.x * 4 + w) * 64; s0 < B; s0 += (int64_t)gridDim.x * 256) {
    float x = s0 + lane < B ? ploss[s0 + lane] : 0.0f;
    for (int ofs = 32; ofs > 0; ofs >>= 1) x += __shfl_xor(x, ofs);
    t += (double)x;
  }
  if (lane == 0 && t != 0.0) atomicAdd(loss, t);
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

__global__ void k_fill_zero(float* x, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    x[i] = 0.0f;
}

hipError_t launch_fill_zero(float* x, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_zero, dim3((n + 255) / 256), dim3(256), 0, s, x, n);
  return hipGetLastError();
}

int mlp_grad_parts(int64_t B) {
  const int64_t g = (B + kGradSamples - 1) / kGradSamples;
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
                           int64_t B, float pos_weight, float* part, float* ploss, double* loss,
                           bool add, hipStream_t s) {
  if (B <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)mlp_grad_parts(B)), dim3(kGradThreads), 0, s, p,
                     X, y, idx, B, 1.0f / (float)B, pos_weight, part, ploss, loss, add ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const float* part, const float* ploss, int64_t B, float* g,
                             double* loss, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kMlpParams + 63) / 64), dim3(256), 0, s, part,
                     ploss, mlp_grad_parts(B), B, g, loss, nullptr, nullptr, nullptr, AdamStep{});
  return hipGetLastError();
}

hipError_t launch_mlp_reduce_step(const float* part, const float* ploss, int64_t B, float* g,
                                  double* loss, float* p, float* m, float* v, int t, float lr,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kMlpParams + 63) / 64), dim3(256), 0, s, part,
                     ploss, mlp_grad_parts(B), B, g, loss, p, m, v, adam_step(t, lr));
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
