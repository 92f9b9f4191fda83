// Refinement classifier: a 64-64-64-1 MLP with GELU, trained in FP32 and
// evaluated in FP16 on the GPU.  Features are the last four rows of a leaf's
// 16 x 16 Chebyshev coefficient array; the logit says "refine".
//
// Parameters: one flat FP32 vector, W1 (64 x 64, [out][in]) at 0, b1 at 4096,
// W2 at 4160, b2 at 8256, w3 at 8320, b3 at 8384 (8385 values).
// GELU is the exact x Phi(x); the loss is the mean binary cross-entropy of
// the logits.  A work-group takes 32 samples.  The 64 x 64 products are
// register-tiled: thread (ts, tu) = (t / 16, t % 16) forms the units tu + 16j
// (j < 4) of the samples 2 ts, 2 ts + 1, reading four contraction indices of
// six rows from LDS (16 bytes each) per 32 multiply-adds; one row per
// multiply-add pair, as before, made the LDS the bound.  Rows are 68 floats
// apart, so the 16 rows a wave reads at once start in different banks.  Every
// sum keeps its order (contraction index ascending from the bias), so the
// results do not depend on the tiling.  A batch of a few thousand boxes is one
// or two rounds of work-groups, bound by their latency (12000 boxes 8.9 us);
// 300000 take 102 us, 49 TFLOP/s of the vector units' 79 without packed
// instructions.  The matrix cores would sum in another order.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cstdint>
#include <string>

#include "vfx_internal.h"

namespace vfx {

namespace {

constexpr int D = 64, S = 32, LDW = D + 4;
constexpr int OW1 = 0, OB1 = 4096, OW2 = 4160, OB2 = 8256, OW3 = 8320, OB3 = 8384;
constexpr int NPAR = 8385;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_prime(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// count values (a multiple of 1024) of a 64-column matrix into LDS rows of
// LDW floats, 256 threads; 16-byte loads where the source is aligned for them
__device__ __forceinline__ void load_rows(const float* __restrict__ src, int count, float* dst) {
  if (((uintptr_t)src & 15) == 0) {
    for (int k = 4 * threadIdx.x; k < count; k += 1024)
      *(float4*)(dst + (k >> 6) * LDW + (k & 63)) = *(const float4*)(src + k);
  } else {
    for (int k = threadIdx.x; k < count; k += 256) dst[(k >> 6) * LDW + (k & 63)] = src[k];
  }
}
__device__ __forceinline__ void load_rows(const __half* __restrict__ src, int count, float* dst) {
  if (((uintptr_t)src & 15) == 0) {
    for (int k = 8 * threadIdx.x; k < count; k += 2048) {
      const uint4 v = *(const uint4*)(src + k);
      const __half* h = (const __half*)&v;
      float* d = dst + (k >> 6) * LDW + (k & 63);
      *(float4*)d = make_float4(__half2float(h[0]), __half2float(h[1]), __half2float(h[2]), __half2float(h[3]));
      *(float4*)(d + 4) = make_float4(__half2float(h[4]), __half2float(h[5]), __half2float(h[6]), __half2float(h[7]));
    }
  } else {
    for (int k = threadIdx.x; k < count; k += 256) dst[(k >> 6) * LDW + (k & 63)] = __half2float(src[k]);
  }
}
// the ns <= S samples s0 ..; rows past them are zero
template <class F>
__device__ __forceinline__ void load_samples(const F* __restrict__ X, long s0, int ns, float* dst) {
  if (ns == S) {
    load_rows(X + s0 * D, S * D, dst);
  } else {
    for (int k = threadIdx.x; k < S * D; k += 256)
      dst[(k >> 6) * LDW + (k & 63)] = (k >> 6) < ns ? (float)X[s0 * D + k] : 0.0f;
  }
}

// z[r][j] += sum_i W[tu + 16 j][i] x[2 ts + r][i], i ascending
__device__ __forceinline__ void tile_product(const float* W, const float* x, float z[2][4]) {
  const int ts = threadIdx.x >> 4, tu = threadIdx.x & 15;
#pragma unroll 4
  for (int i = 0; i < D; i += 4) {
    float4 w[4], v[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = *(const float4*)(W + (tu + 16 * j) * LDW + i);
#pragma unroll
    for (int r = 0; r < 2; ++r) v[r] = *(const float4*)(x + (2 * ts + r) * LDW + i);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        z[r][j] += w[j].x * v[r].x;
        z[r][j] += w[j].y * v[r].y;
        z[r][j] += w[j].z * v[r].z;
        z[r][j] += w[j].w * v[r].w;
      }
  }
}

// sum over the 64 units of a sample: v[j] of unit tu + 16 j, halves first
__device__ __forceinline__ float unit_sum(const float v[4]) {
  float s = (v[0] + v[2]) + (v[1] + v[3]);
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 16);
  return s;
}

// forward pass of the 32 samples in x: z1, z2 and a2 of this thread's outputs
// in registers, a1 in LDS; logits of its samples (every lane of the 16)
__device__ __forceinline__ void forward(const float* W1, const float* W2, const float* x, float* a1,
                                        const float* __restrict__ th, float z1[2][4], float z2[2][4], float a2[2][4],
                                        float logit[2]) {
  const int ts = threadIdx.x >> 4, tu = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < 4; ++j) z1[0][j] = z1[1][j] = th[OB1 + tu + 16 * j];
  tile_product(W1, x, z1);
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) a1[(2 * ts + r) * LDW + tu + 16 * j] = gelu(z1[r][j]);
  __syncthreads();
  float w3[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    z2[0][j] = z2[1][j] = th[OB2 + tu + 16 * j];
    w3[j] = th[OW3 + tu + 16 * j];
  }
  tile_product(W2, a1, z2);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a2[r][j] = gelu(z2[r][j]);
      v[j] = a2[r][j] * w3[j];
    }
    logit[r] = unit_sum(v) + th[OB3];
  }
}

__global__ void __launch_bounds__(256) k_mlp_forward(const float* __restrict__ th, const float* __restrict__ X, long B,
                                                     float* __restrict__ logits) {
  __shared__ __attribute__((aligned(16))) float W1[D * LDW], W2[D * LDW], x[S * LDW], a1[S * LDW];
  load_rows(th + OW1, D * D, W1);
  load_rows(th + OW2, D * D, W2);
  for (long s0 = (long)blockIdx.x * S; s0 < B; s0 += (long)gridDim.x * S) {
    const int ns = (int)min((long)S, B - s0);
    load_samples(X, s0, ns, x);
    __syncthreads();
    float z1[2][4], z2[2][4], a2[2][4], lg[2];
    forward(W1, W2, x, a1, th, z1, z2, a2, lg);
    const int ts = threadIdx.x >> 4, r = threadIdx.x & 15;
    if (r < 2 && 2 * ts + r < ns) logits[s0 + 2 * ts + r] = r ? lg[1] : lg[0];
    __syncthreads();
  }
}

// per-tile partial gradient of the mean loss (1/B factor applied here); the
// partials of the tiles are added in tile order by k_mlp_reduce.  A minibatch
// of 1024 is 32 work-groups, so the time is one work-group's: 34.8 us with
// the untiled products.
__global__ void __launch_bounds__(256) k_mlp_grad_tiles(const float* __restrict__ th, const float* __restrict__ X,
                                                        const float* __restrict__ y, long B,
                                                        float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float W1[D * LDW], W2[D * LDW], x[S * LDW], a1[S * LDW];
  __shared__ __attribute__((aligned(16))) float dz1[S * LDW], dz2[S * LDW], sa2[S * LDW];
  __shared__ float ds[S];
  __shared__ float red[4 * D];
  const long s0 = (long)blockIdx.x * S;
  const int ns = (int)min((long)S, B - s0);
  load_rows(th + OW1, D * D, W1);
  load_rows(th + OW2, D * D, W2);
  load_samples(X, s0, ns, x);
  __syncthreads();
  const int t = threadIdx.x, u = t & 63, g = t >> 6, ts = t >> 4, tu = t & 15;
  float z1[2][4], z2[2][4], a2[2][4], lg[2];
  forward(W1, W2, x, a1, th, z1, z2, a2, lg);
  // d loss / d logit of this thread's samples, then dz2
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int s = 2 * ts + r;
    const float d = s < ns ? (1.0f / (1.0f + expf(-lg[r])) - y[s0 + s]) / (float)B : 0.0f;
    if (tu == 0) ds[s] = d;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sa2[s * LDW + tu + 16 * j] = a2[r][j];
      dz2[s * LDW + tu + 16 * j] = d * th[OW3 + tu + 16 * j] * gelu_prime(z2[r][j]);
    }
  }
  __syncthreads();
  float* P = part + (size_t)blockIdx.x * NPAR;
  // dW3, db3
  float gw3 = 0.0f;
  for (int s = g; s < S; s += 4) gw3 += ds[s] * sa2[s * LDW + u];
  red[g * D + u] = gw3;
  // da1 = W2^T dz2, dz1 (outputs as in the forward pass, unit ascending)
  {
    float a[2][4] = {};
#pragma unroll 4
    for (int o = 0; o < D; o += 4) {
      float4 v[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) v[r] = *(const float4*)(dz2 + (2 * ts + r) * LDW + o);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = W2[(o + k) * LDW + tu + 16 * j];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const float d = k == 0 ? v[r].x : k == 1 ? v[r].y : k == 2 ? v[r].z : v[r].w;
#pragma unroll
          for (int j = 0; j < 4; ++j) a[r][j] += w[j] * d;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) dz1[(2 * ts + r) * LDW + tu + 16 * j] = a[r][j] * gelu_prime(z1[r][j]);
  }
  __syncthreads();
  if (t < D) P[OW3 + t] = (red[t] + red[D + t]) + (red[2 * D + t] + red[3 * D + t]);
  if (t == 0) {
    float b = 0.0f;
    for (int s = 0; s < S; ++s) b += ds[s];
    P[OB3] = b;
  }
  if (t >= 128) {  // db2, db1
    const float* dz = t < 192 ? dz2 : dz1;
    float db = 0.0f;
    for (int s = 0; s < S; ++s) db += dz[s * LDW + u];
    P[(t < 192 ? OB2 : OB1) + u] = db;
  }
  // dW2[o][i] = sum_s dz2[s][o] a1[s][i]; dW1[o][i] = sum_s dz1[s][o] x[s][i]:
  // thread (ts, tu) takes the rows 4 ts .. + 3 and the columns tu + 16 j
#pragma unroll
  for (int layer = 0; layer < 2; ++layer) {
    const float* dz = layer == 0 ? dz2 : dz1;
    const float* in = layer == 0 ? a1 : x;
    float acc[4][4] = {};
#pragma unroll 4
    for (int s = 0; s < S; ++s) {
      const float4 d = *(const float4*)(dz + s * LDW + 4 * ts);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = in[s * LDW + tu + 16 * j];
        acc[0][j] += d.x * v;
        acc[1][j] += d.y * v;
        acc[2][j] += d.z * v;
        acc[3][j] += d.w * v;
      }
    }
    const int OW = layer == 0 ? OW2 : OW1;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) P[OW + (4 * ts + r) * D + tu + 16 * j] = acc[r][j];
  }
}

// tiles j even into one sum, odd into another, sixteen loads in flight
__global__ void k_mlp_reduce(int ntiles, const float* __restrict__ part, float* __restrict__ grad) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= NPAR) return;
  float a0 = 0.0f, a1 = 0.0f;
  int j = 0;
  for (; j + 15 < ntiles; j += 16) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = part[(size_t)(j + i) * NPAR + k];
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      a0 += v[i];
      a1 += v[i + 1];
    }
  }
  for (; j + 1 < ntiles; j += 2) {
    a0 += part[(size_t)j * NPAR + k];
    a1 += part[(size_t)(j + 1) * NPAR + k];
  }
  if (j < ntiles) a0 += part[(size_t)j * NPAR + k];
  grad[k] = a0 + a1;
}

__global__ void k_mlp_adam(float* __restrict__ th, const float* __restrict__ grad, float* __restrict__ m,
                           float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= NPAR) return;
  const float gk = grad[k];
  const float mk = b1 * m[k] + (1.0f - b1) * gk;
  const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  th[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

__global__ void k_to_f16(long n, const float* __restrict__ a, __half* __restrict__ h) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    h[i] = __float2half(a[i]);
}

// FP16 inference: weights, inputs and activations FP16 (held in LDS as the
// FP32 of the same value, so no multiply-add converts), products accumulated
// in FP32.  12000 boxes: 57.8 us with a conversion and an LDS read per factor.
__global__ void __launch_bounds__(256) k_mlp_infer_f16(const __half* __restrict__ th, const __half* __restrict__ X,
                                                       long B, float* __restrict__ logits) {
  __shared__ __attribute__((aligned(16))) float W1[D * LDW], W2[D * LDW], x[S * LDW], a1[S * LDW];
  load_rows(th + OW1, D * D, W1);
  load_rows(th + OW2, D * D, W2);
  const int ts = threadIdx.x >> 4, tu = threadIdx.x & 15;
  float b1[4], b2[4], w3[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    b1[j] = __half2float(th[OB1 + tu + 16 * j]);
    b2[j] = __half2float(th[OB2 + tu + 16 * j]);
    w3[j] = __half2float(th[OW3 + tu + 16 * j]);
  }
  const float b3 = __half2float(th[OB3]);
  for (long s0 = (long)blockIdx.x * S; s0 < B; s0 += (long)gridDim.x * S) {
    const int ns = (int)min((long)S, B - s0);
    load_samples(X, s0, ns, x);
    __syncthreads();
    float z[2][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) z[0][j] = z[1][j] = b1[j];
    tile_product(W1, x, z);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a1[(2 * ts + r) * LDW + tu + 16 * j] = __half2float(__float2half(gelu(z[r][j])));
        z[r][j] = b2[j];
      }
    __syncthreads();
    tile_product(W2, a1, z);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = __half2float(__float2half(gelu(z[r][j]))) * w3[j];
      const float s = unit_sum(v);
      if (tu == r && 2 * ts + r < ns) logits[s0 + 2 * ts + r] = s + b3;
    }
    __syncthreads();
  }
}

}  // namespace

int mlp_param_count() { return NPAR; }

int mlp_forward(const float* th, const float* X, long B, float* logits, hipStream_t s) {
  if (B <= 0) return VFX_OK;
  const int grid = (int)std::min<long>((B + S - 1) / S, 2048);
  hipLaunchKernelGGL(k_mlp_forward, dim3(grid), dim3(256), 0, s, th, X, B, logits);
  return hipGetLastError() == hipSuccess ? VFX_OK : VFX_EHIP;
}

long mlp_grad_work(long B) { return ((B + S - 1) / S) * (long)NPAR; }

int mlp_grad(const float* th, const float* X, const float* y, long B, float* grad, float* work, hipStream_t s) {
  if (B <= 0) return VFX_EINVAL;
  const int ntiles = (int)((B + S - 1) / S);
  hipLaunchKernelGGL(k_mlp_grad_tiles, dim3(ntiles), dim3(256), 0, s, th, X, y, B, work);
  hipLaunchKernelGGL(k_mlp_reduce, dim3((NPAR + 255) / 256), dim3(256), 0, s, ntiles, work, grad);
  return hipGetLastError() == hipSuccess ? VFX_OK : VFX_EHIP;
}

int mlp_adam(float* th, const float* grad, float* m, float* v, int step, float lr, float b1, float b2, float eps,
             hipStream_t s) {
  if (step < 1) return VFX_EINVAL;
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_mlp_adam, dim3((NPAR + 255) / 256), dim3(256), 0, s, th, grad, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? VFX_OK : VFX_EHIP;
}

int mlp_to_f16(const float* a, uint16_t* h, long n, hipStream_t s) {
  if (n <= 0) return VFX_OK;
  const int grid = (int)std::min<long>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_to_f16, dim3(grid), dim3(256), 0, s, n, a, (__half*)h);
  return hipGetLastError() == hipSuccess ? VFX_OK : VFX_EHIP;
}

int mlp_infer_f16(const uint16_t* th, const uint16_t* X, long B, float* logits, hipStream_t s) {
  if (B <= 0) return VFX_OK;
  const int grid = (int)std::min<long>((B + S - 1) / S, 2048);
  hipLaunchKernelGGL(k_mlp_infer_f16, dim3(grid), dim3(256), 0, s, (const __half*)th, (const __half*)X, B, logits);
  return hipGetLastError() == hipSuccess ? VFX_OK : VFX_EHIP;
}

}  // namespace vfx
