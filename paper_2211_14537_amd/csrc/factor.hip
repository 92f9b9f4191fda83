// Plan stage on the GPU: the per-cut-leaf least-squares operators
// P_i = A_{X^I,G}^+ (Section 3.2: the least-squares fit on the interior
// stencil points; the paper factors each cut square by QR), for every cut
// leaf at once, one work-group per cut leaf, in FP64:
//   1. M = A[X^I, :] (N_I x N_G), column-major in a scratch buffer;
//   2. Householder QR of M, reflectors kept below the diagonal;
//   3. one-sided Jacobi SVD of B = R^T (N_G x r, r = min(N_I, N_G)) in LDS,
//      round-robin pairs, rotations accumulated in W (r x r);
//   4. pinv(R) = B diag(1/sigma^2) W^T, singular values below 1e-13 sigma_max
//      dropped (the minimum-norm solution when N_I < N_G);
//   5. P_i = pinv(R) Q^T, formed as Q [pinv(R)^T; 0] by applying the
//      reflectors in reverse order, written as P_i (N_G x N_I row-major).
// The whole is a chain of short steps (about ten Jacobi sweeps of 65 rounds,
// 66 reflectors twice), so its time is latency.  A work-group has 36 groups
// of 16 lanes: a round's 33 rotations run side by side, one per group, and a
// reflector is applied to 36 columns at once, with the 16-lane sums formed by
// DPP rotations inside a row of the wave.  730 cut leaves: 29.4 ms with one
// wave per pair and per column (four of each at a time).  The sums keep the
// order of a 64-lane butterfly over elements 64 apart, in which they were
// defined first: P_i has entries up to cond(A_I), so another order would
// change f^e by that much rounding.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>

#include "vfx_internal.h"

#define VFX_HIP(call)                                                          \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) {                                                    \
      err = std::string(#call) + ": " + hipGetErrorString(e_);                 \
      return VFX_EHIP;                                                         \
    }                                                                          \
  } while (0)

namespace vfx {

namespace {

constexpr int kG = 66;          // support points handled (stencil degree <= 10)
constexpr int LDB = kG + 1;     // LDS column stride
constexpr double kCut = 1e-13;  // relative singular-value cut-off
constexpr int kMaxSweeps = 40;

constexpr int kThreads = 576;   // 36 groups of 16 lanes, nine waves
constexpr int kGroups = kThreads / 16;

__device__ __forceinline__ double wsum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// v of the lane N further round the row of 16
template <int N>
__device__ __forceinline__ double ror(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, 0x120 + N, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), 0x120 + N, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// sum over a group of 16 lanes, lane l holding the partial sums of the lanes
// l, l + 16, l + 32, l + 48 of a wave: the butterfly over distances 32, 16
// (here inside the lane), 8, 4, 2, 1 (after each step the sums repeat with
// that period, so a rotation fetches the partner's).  Products that enter it
// are rounded first, as they were before the exchange of a butterfly.
__device__ __forceinline__ double gsum(double v0, double v1, double v2, double v3) {
#pragma clang fp contract(off)
  double v = (v0 + v2) + (v1 + v3);
  v += ror<8>(v);
  v += ror<4>(v);
  v += ror<2>(v);
  v += ror<1>(v);
  return v;
}

// sum over the first 256 threads; red: 4 doubles of LDS
__device__ double block_sum(double v, double* red) {
  v = wsum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0 && w < 4) red[w] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// the reflector v (elements j .. m-1 of column M_j, factor tau) applied to a
// column x by a group of 16 lanes: x -= tau (v . x) v
constexpr int kRows = 32;  // elements per lane held in registers (m - j <= 16 kRows)
__device__ __forceinline__ void reflect(const double* __restrict__ v, double* __restrict__ x, int j, int m, double tau,
                                        int l) {
  const int len = m - j;
  if (len <= 16 * kRows) {
    // x stays in registers, v is read twice; chunks of 8 x 16 elements
    const double* vp = v + j + l;
    double* xp = x + j + l;
    double b[kRows], s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k0 = 0; k0 < kRows; k0 += 8)
      if (16 * k0 < len) {
        double a[8];
        const int left = len - l - 16 * k0;  // element k of the chunk exists if 16 k < left
        if (16 * k0 + 128 <= len) {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            a[k] = vp[16 * (k0 + k)];
            b[k0 + k] = xp[16 * (k0 + k)];
          }
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            a[k] = 16 * k < left ? vp[16 * (k0 + k)] : 0.0;
            b[k0 + k] = 16 * k < left ? xp[16 * (k0 + k)] : 0.0;
          }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k & 3] = __builtin_fma(a[k], b[k0 + k], s[k & 3]);
      }
    const double d = gsum(s[0], s[1], s[2], s[3]) * tau;
#pragma unroll
    for (int k0 = 0; k0 < kRows; k0 += 8)
      if (16 * k0 < len) {
        const int left = len - l - 16 * k0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (16 * k < left) xp[16 * (k0 + k)] = __builtin_fma(-d, vp[16 * (k0 + k)], b[k0 + k]);
      }
  } else {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = j + l, k = 0; i < m; i += 16, ++k) {
      if ((k & 3) == 0) s[0] = __builtin_fma(v[i], x[i], s[0]);
      if ((k & 3) == 1) s[1] = __builtin_fma(v[i], x[i], s[1]);
      if ((k & 3) == 2) s[2] = __builtin_fma(v[i], x[i], s[2]);
      if ((k & 3) == 3) s[3] = __builtin_fma(v[i], x[i], s[3]);
    }
    const double d = gsum(s[0], s[1], s[2], s[3]) * tau;
    for (int i = j + l; i < m; i += 16) x[i] = __builtin_fma(-d, v[i], x[i]);
  }
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) k_factor(int nG, const int* __restrict__ pinv_ptr,
                                                     const uint16_t* __restrict__ pinv_idx,
                                                     const double* __restrict__ A, double* __restrict__ ws,
                                                     double* __restrict__ Pout) {
  __shared__ double sB[kG * LDB];  // B = R^T, column i at sB[i * LDB]
  __shared__ double sW[kG * LDB];  // rotations, column i at sW[i * LDB]
  __shared__ double tau[kG], rdiag[kG], sig2[kG];
  __shared__ double red[4];
  __shared__ double s_off[kThreads / 64];
  const int c = blockIdx.x;
  const int off = pinv_ptr[c], m = pinv_ptr[c + 1] - off;
  if (m == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int grp = tid >> 4, l = tid & 15;
  double* M = ws + (size_t)off * nG;    // column j at M + j*m
  double* Z = Pout + (size_t)off * nG;  // column t at Z + t*m (= row t of P_i)
  const int r = min(m, nG);
  // 1. gather
  for (int e = tid; e < m * nG; e += blockDim.x) {
    const int i = e % m, j = e / m;
    M[(size_t)j * m + i] = A[(size_t)pinv_idx[off + i] * nG + j];
  }
  __syncthreads();
  // 2. Householder QR
  for (int j = 0; j < r; ++j) {
    double part = 0.0;
    if (tid < 256)
      for (int i = j + tid; i < m; i += 256) part += M[(size_t)j * m + i] * M[(size_t)j * m + i];
    const double nrm2 = block_sum(part, red);
    if (tid == 0) {
      const double x0 = M[(size_t)j * m + j];
      const double nrm = sqrt(nrm2);
      const double alpha = x0 >= 0 ? -nrm : nrm;
      const double v0 = x0 - alpha;
      const double vn2 = nrm2 - x0 * x0 + v0 * v0;
      tau[j] = vn2 > 0 ? 2.0 / vn2 : 0.0;
      rdiag[j] = nrm2 > 0 ? alpha : 0.0;
      M[(size_t)j * m + j] = v0;
    }
    __syncthreads();
    const double tj = tau[j];
    for (int cc = j + 1 + grp; cc < nG; cc += kGroups) reflect(M + (size_t)j * m, M + (size_t)cc * m, j, m, tj, l);
    __syncthreads();
  }
  // 3. B = R^T (column i of B = row i of R), W = I
  for (int e = tid; e < kG * kG; e += blockDim.x) {
    const int i = e / kG, t = e % kG;
    double b = 0.0;
    if (i < r && t < nG) b = (t == i) ? rdiag[i] : (t > i ? M[(size_t)t * m + i] : 0.0);
    sB[i * LDB + t] = b;
    sW[i * LDB + t] = (i == t && i < r) ? 1.0 : 0.0;
  }
  __syncthreads();
  // one-sided Jacobi on the r columns of B (round-robin pairs)
  const int np = (r + 1) & ~1;  // players, even
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    double offmax = 0.0;
    for (int rd = 0; rd < np - 1; ++rd) {
      // pair grp of the round: lane l holds the elements l + 16k (k < 4) and,
      // l < 2, 64 + l of both columns (entries past nG or r are zero)
      const int a = grp == 0 ? 0 : 1 + (rd + grp - 1) % (np - 1);
      const int b = 1 + (rd + np - 1 - grp - 1) % (np - 1);
      if (grp < np / 2 && a < r && b < r) {
        double *Ba = sB + a * LDB + l, *Bb = sB + b * LDB + l, *Wa = sW + a * LDB + l, *Wb = sW + b * LDB + l;
        double x[5], y[5], p[4], q[4], g[4];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          const bool ok = k < 4 || l < kG - 64;
          x[k] = ok ? Ba[16 * k] : 0.0;
          y[k] = ok ? Bb[16 * k] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          p[k] = __builtin_fma(x[k], x[k], 0.0);  // rounded products
          q[k] = __builtin_fma(y[k], y[k], 0.0);
          g[k] = __builtin_fma(x[k], y[k], 0.0);
        }
        p[0] = __builtin_fma(x[4], x[4], p[0]);
        q[0] = __builtin_fma(y[4], y[4], q[0]);
        g[0] = __builtin_fma(x[4], y[4], g[0]);
        const double al = gsum(p[0], p[1], p[2], p[3]), be = gsum(q[0], q[1], q[2], q[3]);
        const double ga = gsum(g[0], g[1], g[2], g[3]);
        if (!(ga == 0.0 || al == 0.0 || be == 0.0)) {
          const double rel = fabs(ga) / sqrt(al * be);
          offmax = fmax(offmax, rel);
          if (!(rel < 1e-16)) {
            const double zeta = (be - al) / (2.0 * ga);
            const double tt = (zeta >= 0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
            const double cs = 1.0 / sqrt(1.0 + tt * tt), sn = cs * tt;
#pragma unroll
            for (int k = 0; k < 5; ++k)
              if (k < 4 || l < kG - 64) {
                Ba[16 * k] = cs * x[k] - sn * y[k];
                Bb[16 * k] = sn * x[k] + cs * y[k];
                const double u = Wa[16 * k], v = Wb[16 * k];
                Wa[16 * k] = cs * u - sn * v;
                Wb[16 * k] = sn * u + cs * v;
              }
          }
        }
      }
      __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1) offmax = fmax(offmax, __shfl_xor(offmax, o, 64));
    if (lane == 0) s_off[w] = offmax;
    __syncthreads();
    double om = s_off[0];
    for (int k = 1; k < kThreads / 64; ++k) om = fmax(om, s_off[k]);
    __syncthreads();
    if (om < 1e-15) break;
  }
  // 4. squared singular values, cut-off
  for (int i = w; i < r; i += kThreads / 64) {
    double s = 0.0;
    for (int t = lane; t < nG; t += 64) s += sB[i * LDB + t] * sB[i * LDB + t];
    s = wsum(s);
    if (lane == 0) sig2[i] = s;
  }
  __syncthreads();
  double smax = 0.0;
  for (int i = 0; i < r; ++i) smax = fmax(smax, sig2[i]);
  // X = pinv(R)^T (r x nG): X[k][t] = sum_i W[k][i] B[t][i] / sig2[i] -> Z rows k < r
  for (int e = tid; e < nG * m; e += blockDim.x) {
    const int k = e % m, t = e / m;
    double x = 0.0;
    if (k < r)
      for (int i = 0; i < r; ++i)
        if (sig2[i] > kCut * kCut * smax) x += sW[i * LDB + k] * sB[i * LDB + t] / sig2[i];
    Z[(size_t)t * m + k] = x;
  }
  __syncthreads();
  // 5. Z = H_0 ... H_{r-1} Z
  for (int j = r - 1; j >= 0; --j) {
    const double tj = tau[j];
    for (int t = grp; t < nG; t += kGroups) reflect(M + (size_t)j * m, Z + (size_t)t * m, j, m, tj, l);
    __syncthreads();
  }
}

}  // namespace

int factor_gpu(Plan* p, hipStream_t s, std::string& err) {
  const HostPlan& H = p->H;
  DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  if (T.nG > kG) {
    err = "the GPU factorisation supports at most 66 support points (stencil degree <= 10)";
    return VFX_EINVAL;
  }
  if (H.ncut == 0) {
    D.factored = true;
    return VFX_OK;
  }
  const size_t nv = (size_t)H.pinv_ptr[H.ncut] * T.nG;
  if (!D.fac_ws) VFX_HIP(hipMalloc((void**)&D.fac_ws, sizeof(double) * nv));
  hipLaunchKernelGGL(k_factor, dim3(H.ncut), dim3(kThreads), 0, s, T.nG, D.pinv_ptr, D.pinv_idx, p->ctx->D.A, D.fac_ws,
                     D.pinv_val);
  VFX_HIP(hipGetLastError());
  D.factored = true;
  return VFX_OK;
}

}  // namespace vfx
