// Training of the child-ordering network: loss, backpropagation and Adam, on
// the GPU.  One block takes 64 samples of a minibatch: eight waves share the
// units of every layer (a lane per sample, weights in LDS), then the parameters'
// gradient sums over the block's samples, in a fixed order, and write one partial
// row; a second kernel adds the rows in block order (deterministic), divides by
// the number of labelled samples and applies the update.
//
// Network and parameter order as in policy.h.  In bfloat16 mode the inputs,
// the weights and the hidden activations are rounded to bfloat16 as in
// inference, sums stay fp32 and gradients pass straight through the roundings
// to the fp32 master weights.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "policy.h"

namespace ccs {

constexpr int kMlpBlock = 64;     // samples of a block; threads of a reduction block
constexpr int kMlpThreads = 512;  // eight waves per gradient block
constexpr int kMlpRow = 68;       // words of an LDS row of 64 samples: rows 4 banks apart

__device__ __forceinline__ float bf16_value(float x) { return __uint_as_float(bf16_bits(x) << 16); }

// Minibatch sample k of the affine permutation (a * pos + c) mod n, gcd(a, n) = 1.
// inv = floor((2^64 - 1) / n): the quotient estimate floor(x inv / 2^64) is at most
// 2 below the true one (x inv / 2^64 is less than 1 + 1/n below x / n).
__device__ __forceinline__ uint32_t perm_index(uint64_t pos, uint64_t a, uint64_t c, uint32_t n, uint64_t inv) {
  if (pos >= n) pos %= n;
  const uint64_t x = a * pos + c;
  uint64_t r = x - __umul64hi(x, inv) * n;
  if (r >= n) r -= n;
  if (r >= n) r -= n;
  return (uint32_t)r;
}

__device__ __forceinline__ float comp(const float4& v, int k) { return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w; }

// A tile of weight gradients: rows d0 + dstep i (i < 2) of the deltas by rows a0 +
// astep j (j < 4) of the activations, each summed over the 64 samples in order.
__device__ __forceinline__ void grad_tile(const float (*del)[kMlpRow], const float (*act)[kMlpRow], int d0, int dstep,
                                          int a0, int astep, float* out, int out0, int out_d, int out_a) {
  float g[2][4] = {};
#pragma unroll 4
  for (int t = 0; t < kMlpBlock / 4; ++t) {
    float4 d[2], a[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) d[i] = *reinterpret_cast<const float4*>(&del[d0 + dstep * i][4 * t]);
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = *reinterpret_cast<const float4*>(&act[a0 + astep * j][4 * t]);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) g[i][j] = fmaf(comp(d[i], k), comp(a[j], k), g[i][j]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) out[out0 + out_d * i + out_a * j] = g[i][j];
}

__device__ __forceinline__ float row_sum(const float* row) {
  float g = 0.0f;
#pragma unroll
  for (int t = 0; t < kMlpBlock / 4; ++t) {
    const float4 v = *reinterpret_cast<const float4*>(&row[4 * t]);
    g += v.x;
    g += v.y;
    g += v.z;
    g += v.w;
  }
  return g;
}

// What bounds it: the chain of sums (16 + 32 + 32 + 32 + 64 terms, whose order is
// the result's) and the latency of the row and weight loads, at 128 blocks of a
// batch of 8192.  Wave w holds units 4w .. 4w + 3 of either hidden layer, so a lane
// runs four chains at once where one thread per sample ran 32, and the gradient
// sums take 2 x 4 tiles of parameters per lane (six 16-byte LDS reads for 32 fused
// multiply-adds; 8 rows of a tile column 4 banks apart).  8192 rows: 45 -> 9.5 us.
__global__ __launch_bounds__(kMlpThreads) void k_mlp_grad(const float* __restrict__ theta, const float* __restrict__ X,
                                                          const uint8_t* __restrict__ Y, uint32_t n, uint32_t batch,
                                                          uint64_t pos0, uint64_t pa, uint64_t pc, uint64_t inv,
                                                          int bf16, float* __restrict__ partial,
                                                          float* __restrict__ lossp) {
  __shared__ __align__(16) float w[kPolicyParams];
  __shared__ __align__(16) float act[80][kMlpRow];  // x (16), h1 (32), h2 (32); a row over the samples
  __shared__ __align__(16) float del[68][kMlpRow];  // d1 (32), d2 (32), d3 (4): gradients at the pre-activations
  __shared__ __align__(16) float red[2][kMlpRow];
  __shared__ float zs[4][kMlpBlock];
  const int tid = threadIdx.x, s = tid & 63, wv = tid >> 6;
  const uint32_t k = blockIdx.x * kMlpBlock + s;
  uint32_t label = 255u;
  float x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = 0.0f;
  if (k < batch) {
    const uint32_t row = perm_index(pos0 + k, pa, pc, n, inv);
    label = Y[row];
    const float4* xr = reinterpret_cast<const float4*>(X + (size_t)row * 16);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = xr[q];
      x[4 * q] = v.x;
      x[4 * q + 1] = v.y;
      x[4 * q + 2] = v.z;
      x[4 * q + 3] = v.w;
    }
  }
  for (int p = tid; p < kPolicyParams; p += kMlpThreads) {
    const bool is_w = p < kPolicyB1 || (p >= kPolicyW2 && p < kPolicyB2) || (p >= kPolicyW3 && p < kPolicyB3);
    const float v = theta[p];
    w[p] = (bf16 && is_w) ? bf16_value(v) : v;
  }
  const bool lab = label < 4u;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    if (bf16) x[q] = bf16_value(x[q]);
    x[q] = lab ? x[q] : 0.0f;
    if ((q >> 1) == wv) act[q][s] = x[q];
  }
  __syncthreads();
  const int u0 = 4 * wv;  // this wave's units
  bool m1[4], m2[4];      // ReLU masks
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float4* wr = reinterpret_cast<const float4*>(w + kPolicyW1 + (u0 + j) * 16);
    float a = w[kPolicyB1 + u0 + j];
#pragma unroll
    for (int q = 0; q < 16; ++q) a = fmaf(comp(wr[q >> 2], q & 3), x[q], a);
    m1[j] = lab && a > 0.0f;
    const float h = fmaxf(a, 0.0f);
    act[16 + u0 + j][s] = lab ? (bf16 ? bf16_value(h) : h) : 0.0f;
  }
  __syncthreads();
  {
    float a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = w[kPolicyB2 + u0 + j];
#pragma unroll
    for (int q4 = 0; q4 < 8; ++q4) {
      float h[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = act[16 + 4 * q4 + q][s];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 wr = *reinterpret_cast<const float4*>(w + kPolicyW2 + (u0 + j) * 32 + 4 * q4);
#pragma unroll
        for (int q = 0; q < 4; ++q) a[j] = fmaf(comp(wr, q), h[q], a[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      m2[j] = lab && a[j] > 0.0f;
      const float h = fmaxf(a[j], 0.0f);
      act[48 + u0 + j][s] = lab ? (bf16 ? bf16_value(h) : h) : 0.0f;
    }
  }
  __syncthreads();
  if (wv < 4) {
    float a = w[kPolicyB3 + wv];
#pragma unroll
    for (int q4 = 0; q4 < 8; ++q4) {
      const float4 wr = *reinterpret_cast<const float4*>(w + kPolicyW3 + wv * 32 + 4 * q4);
#pragma unroll
      for (int q = 0; q < 4; ++q) a = fmaf(comp(wr, q), act[48 + 4 * q4 + q][s], a);
    }
    zs[wv][s] = a;
  }
  __syncthreads();
  float loss = 0.0f;
  float d3[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (lab) {
    float z[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) z[o] = zs[o][s];
    const float zm = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
    float e[4], se = 0.0f;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      e[o] = expf(z[o] - zm);
      se += e[o];
    }
    const float zy = label == 0 ? z[0] : label == 1 ? z[1] : label == 2 ? z[2] : z[3];
    loss = logf(se) + zm - zy;
#pragma unroll
    for (int o = 0; o < 4; ++o) d3[o] = e[o] / se - (label == (uint32_t)o ? 1.0f : 0.0f);
  }
  // backward to the pre-activations
  if (wv == 0) {
    red[0][s] = loss;
    red[1][s] = lab ? 1.0f : 0.0f;
#pragma unroll
    for (int o = 0; o < 4; ++o) del[64 + o][s] = d3[o];
  }
  {
    float g[4] = {};
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const float4 wr = *reinterpret_cast<const float4*>(w + kPolicyW3 + o * 32 + u0);
#pragma unroll
      for (int j = 0; j < 4; ++j) g[j] = fmaf(comp(wr, j), d3[o], g[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) del[32 + u0 + j][s] = m2[j] ? g[j] : 0.0f;
  }
  __syncthreads();
  {
    float g[4] = {};
#pragma unroll 8
    for (int u = 0; u < 32; ++u) {
      const float4 wr = *reinterpret_cast<const float4*>(w + kPolicyW2 + u * 32 + u0);
      const float d2 = del[32 + u][s];
#pragma unroll
      for (int j = 0; j < 4; ++j) g[j] = fmaf(comp(wr, j), d2, g[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) del[u0 + j][s] = m1[j] ? g[j] : 0.0f;
  }
  __syncthreads();
  // parameter gradients summed over the block's samples in sample order
  float* out = partial + (size_t)blockIdx.x * kPolicyParams;
  if (wv < 2) {  // W2: 16 x 8 tiles
    const int d = tid >> 3, a = tid & 7;
    grad_tile(del, act, 32 + d, 16, 16 + a, 8, out, kPolicyW2 + d * 32 + a, 16 * 32, 8);
  } else if (wv == 2) {  // W1: 16 x 4 tiles
    const int d = s >> 2, a = s & 3;
    grad_tile(del, act, d, 16, a, 4, out, kPolicyW1 + d * 16 + a, 16 * 16, 4);
  } else if (wv == 3) {  // W3: 2 x 8 tiles
    const int d = s >> 3, a = s & 7;
    if (s < 16) grad_tile(del, act, 64 + d, 2, 48 + a, 8, out, kPolicyW3 + d * 32 + a, 2 * 32, 8);
  } else if (wv == 4) {  // b1, b2
    out[s < 32 ? kPolicyB1 + s : kPolicyB2 + s - 32] = row_sum(del[s]);
  } else if (wv == 5) {  // b3, loss and labelled count
    if (s < 4) out[kPolicyB3 + s] = row_sum(del[64 + s]);
    else if (s < 6) lossp[2 * blockIdx.x + (s - 4)] = row_sum(red[s - 4]);
  }
}

// Sum of every kStride-th value from v in order, kBatch loads in flight.
template <int kBatch>
__device__ __forceinline__ float ordered_sum(const float* __restrict__ v, size_t stride, uint32_t count) {
  float g = 0.0f;
  uint32_t b = 0;
  for (; b + kBatch <= count; b += kBatch) {
    float x[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) x[q] = v[(size_t)(b + q) * stride];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) g += x[q];
  }
  for (; b < count; ++b) g += v[(size_t)b * stride];
  return g;
}

// Labelled samples of all blocks.  Counts are whole numbers of at most 64 a block,
// so up to 2^18 blocks their fp32 sum is exact in any order and the wave adds them
// in parallel; beyond, in block order as ever.
__device__ __forceinline__ float labelled_count(const float* __restrict__ lossp, uint32_t nblk) {
  if (nblk > (1u << 18)) return ordered_sum<16>(lossp + 1, 2, nblk);
  float c = 0.0f;
  for (uint32_t b = threadIdx.x & 63; b < nblk; b += 64) c += lossp[2 * (size_t)b + 1];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) c += __shfl_xor(c, d);
  return c;
}

// The rows' sums are serial chains over the blocks (their order is the result's), one
// parameter a lane; what a wave waits for is the loads, of which 64 are in flight
// (one at a time: 31 us for 128 rows, now 4.3 us).
constexpr int kReduceBatch = 64;

// Mean loss by the first lane of the block behind the parameters' blocks.
__device__ __forceinline__ void reduce_loss(const float* __restrict__ lossp, uint32_t nblk, float cnt,
                                            float* __restrict__ loss_out) {
  if (threadIdx.x == 0 && loss_out) *loss_out = ordered_sum<kReduceBatch>(lossp, 2, nblk) / fmaxf(cnt, 1.0f);
}

constexpr int kParamBlocks = (kPolicyParams + kMlpBlock - 1) / kMlpBlock;

__global__ __launch_bounds__(kMlpBlock) void k_mlp_reduce(const float* __restrict__ partial,
                                                          const float* __restrict__ lossp, uint32_t nblk,
                                                          float* __restrict__ grad, float* __restrict__ loss_out) {
  const float cnt = labelled_count(lossp, nblk);
  if (blockIdx.x == kParamBlocks) {
    reduce_loss(lossp, nblk, cnt, loss_out);
    return;
  }
  const int p = blockIdx.x * kMlpBlock + threadIdx.x;
  if (p >= kPolicyParams) return;
  grad[p] = ordered_sum<kReduceBatch>(partial + p, kPolicyParams, nblk) / fmaxf(cnt, 1.0f);
}

// Adam with bias corrections c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ __launch_bounds__(kMlpBlock) void k_mlp_adam(float* __restrict__ theta, float* __restrict__ m,
                                                        float* __restrict__ v, const float* __restrict__ partial,
                                                        const float* __restrict__ lossp, uint32_t nblk, float lr,
                                                        float beta1, float beta2, float eps, float c1, float c2,
                                                        float* __restrict__ loss_out) {
  const float cnt = labelled_count(lossp, nblk);
  if (blockIdx.x == kParamBlocks) {
    reduce_loss(lossp, nblk, cnt, loss_out);
    return;
  }
  const int p = blockIdx.x * kMlpBlock + threadIdx.x;
  if (p >= kPolicyParams) return;
  const float g = ordered_sum<kReduceBatch>(partial + p, kPolicyParams, nblk) / fmaxf(cnt, 1.0f);
  const float mm = beta1 * m[p] + (1.0f - beta1) * g;
  const float vv = beta2 * v[p] + (1.0f - beta2) * g * g;
  m[p] = mm;
  v[p] = vv;
  theta[p] -= lr * (mm * c1) / (sqrtf(vv * c2) + eps);
}

__global__ void k_fill(float* __restrict__ p, uint32_t n, float value) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

hipError_t launch_mlp_grad(const float* theta, const float* X, const uint8_t* Y, uint32_t n, uint32_t batch,
                           uint64_t pos0, uint64_t pa, uint64_t pc, int bf16, float* partial, float* lossp,
                           hipStream_t stream) {
  const uint32_t nblk = (batch + kMlpBlock - 1) / kMlpBlock;
  hipLaunchKernelGGL(k_mlp_grad, dim3(nblk), dim3(kMlpThreads), 0, stream, theta, X, Y, n, batch, pos0, pa, pc,
                     ~0ull / n, bf16, partial, lossp);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const float* partial, const float* lossp, uint32_t nblk, float* grad, float* loss,
                             hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kParamBlocks + 1), dim3(kMlpBlock), 0, stream,
                     partial, lossp, nblk, grad, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* theta, float* m, float* v, const float* partial, const float* lossp, uint32_t nblk,
                           float lr, float beta1, float beta2, float eps, float c1, float c2, float* loss,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_adam, dim3(kParamBlocks + (loss ? 1 : 0)), dim3(kMlpBlock), 0, stream,
                     theta, m, v, partial, lossp, nblk, lr, beta1, beta2, eps, c1, c2, loss);
  return hipGetLastError();
}

hipError_t launch_fill(float* p, uint32_t n, float value, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3((n + 255) / 256), dim3(256), 0, stream, p, n, value);
  return hipGetLastError();
}

// Gradient scratch of the entry point that allocates nothing: partial rows of
// kGradScratchBlocks blocks, then their (loss, count) pairs.  One copy per device,
// held until the process ends; every call on a device shares it.
static __device__ __align__(256) float scratch[kGradScratchBlocks * (kPolicyParams + 2)];

hipError_t grad_scratch(float** partial, float** lossp) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* base[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!base[dev]) {
    // the array's address on the current device (its host-side name is not a device address)
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    base[dev] = static_cast<float*>(p);
  }
  *partial = base[dev];
  *lossp = base[dev] + (size_t)kGradScratchBlocks * kPolicyParams;
  return hipSuccess;
}

}  // namespace ccs
