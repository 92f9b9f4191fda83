// Plan stage on the GPU: the per-cut-leaf least-squares operators
// P_i = A_{X^I,G}^+ (Section 3.2: the least-squares fit on the interior
// stencil points; the paper factors each cut square by QR), for every cut
// leaf at once, one work-group per cut leaf, in FP64:
//   k_qr      M = A[X^I, :] (N_I x N_G) and its Householder QR, reflectors
//             kept below the diagonal;
//   k_jacobi  one-sided Jacobi SVD of B = R^T (N_G x r, r = min(N_I, N_G)) in
//             LDS, round-robin pairs, rotations accumulated in W (r x r);
//             pinv(R) = B diag(1/sigma^2) W^T, singular values below
//             1e-13 sigma_max dropped (the minimum-norm solution when
//             N_I < N_G);
//   k_apply   P_i = pinv(R) Q^T, formed as Q [pinv(R)^T; 0] by applying the
//             reflectors in reverse order, written as P_i (N_G x N_I
//             row-major).
// Each is a chain of short steps (66 reflectors, about ten sweeps of 65
// rounds), so its time is latency, and the matrices of all cut leaves
// together (up to 0.5 MB each with the scratch) do not stay in the caches:
// with them in memory the reflectors took 5.4 of 9.5 ms for 730 cut leaves.
// k_qr and k_apply therefore hold their matrix in registers (36 groups of 16
// lanes, two columns per group, up to 480 rows) and pass one reflector at a
// time through LDS; k_jacobi runs a round's 33 rotations side by side, 16
// lanes per pair (8 lanes: 6.2 ms, 4 lanes: 7.3 ms).  730 cut leaves: 0.77 +
// 5.6 + 0.56 ms.
// (One wave per pair and column, four at a time, took 29.4 ms.)
// The sums keep the order of a 64-lane butterfly over elements 64 apart, in
// which they were defined first: P_i has entries up to cond(A_I), so another
// order would change f^e by that much rounding.
#include <hip/hip_runtime.h>

#include <algorithm>
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
constexpr int kMaxX = 648;      // stencil points at most (K, Kbar <= 16, degree <= 15)

// per cut leaf in the scratch past the matrices: tau, rdiag
constexpr int kAux = 2 * kG;

__device__ __forceinline__ double wsum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over a group of 16 lanes of which each holds the partial sums of four
// lanes of a wave 16 apart: the butterfly over distances 32, 16 (here inside
// the lane), 8, 4, 2, 1 (after each step the sums repeat with that period, so
// a rotation of the row fetches the partner's, wherever in the row the order
// starts).  Products that enter it are rounded first, as they were before the
// exchange of a butterfly.
__device__ __forceinline__ double gsum(double v0, double v1, double v2, double v3) {
#pragma clang fp contract(off)
  double v = (v0 + v2) + (v1 + v3);
  v += dpp<0x128>(v);
  v += dpp<0x124>(v);
  v += dpp<0x122>(v);
  v += dpp<0x121>(v);
  return v;
}

// sum over the first 256 threads; red: 4 doubles of LDS
__device__ double block_sum(double v, double* red) {
  v = wsum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0 && w < 4) red[w] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// The reflector v (LDS, zero above row j, factor tau) applied to the column
// whose rows l + 16k this lane holds: x -= tau (v . x) v.  The sums start at
// row j, so the partial sums of the lane rotate with it.
template <int RK>
__device__ __forceinline__ void reflect(const double* v, double x[RK], int j, double tau, int l) {
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  asm volatile("" : "+v"(l));
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    s[k & 3] = __builtin_fma(v[l + 16 * k], x[k], s[k & 3]);
    if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // few elements of v in registers
  }
  const int first = (j >> 4) + (l < (j & 15) ? 1 : 0);
  if (first & 1) {
    const double t = s[0];
    s[0] = s[1], s[1] = s[2], s[2] = s[3], s[3] = t;
  }
  if (first & 2) {
    double t = s[0];
    s[0] = s[2], s[2] = t;
    t = s[1];
    s[1] = s[3], s[3] = t;
  }
  const double d = gsum(s[0], s[1], s[2], s[3]) * tau;
  asm volatile("" : "+v"(l));  // v is read again: held, it would not fit beside x
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    x[k] = __builtin_fma(-d, v[l + 16 * k], x[k]);
    if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);
  }
}

template <int RK>
__global__ void __launch_bounds__(kThreads) k_qr(int nG, const int* __restrict__ pinv_ptr,
                                                 const uint16_t* __restrict__ pinv_idx, const double* __restrict__ A,
                                                 double* __restrict__ ws, double* __restrict__ aux) {
  __shared__ double sV[2][16 * RK];
  __shared__ double red[4];
  __shared__ double s_tau;
  const int c = blockIdx.x;
  const int off = pinv_ptr[c], m = pinv_ptr[c + 1] - off;
  if (m == 0) return;
  const int tid = threadIdx.x, grp = tid >> 4, l = tid & 15;
  const int r = min(m, nG);
  double* M = ws + (size_t)off * nG;  // column j at M + j*m
  aux += (size_t)c * kAux;
  // columns grp and grp + 36 of M, rows l + 16k
  double x[2][RK];
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    const int i = l + 16 * k;
    const size_t row = i < m ? (size_t)pinv_idx[off + i] * nG : 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) x[u][k] = i < m && grp + kGroups * u < nG ? A[row + grp + kGroups * u] : 0.0;
  }
  for (int j = 0; j < r; ++j) {
    double* v = sV[j & 1];
    const int own = j >= kGroups ? 1 : 0;
    if (grp == j - kGroups * own) {
#pragma unroll
      for (int k = 0; k < RK; ++k) v[l + 16 * k] = l + 16 * k < j ? 0.0 : (own ? x[1][k] : x[0][k]);
    }
    __syncthreads();
    double part = 0.0;
    if (tid < 256)
      for (int i = j + tid; i < m; i += 256) part = __builtin_fma(v[i], v[i], part);
    const double nrm2 = block_sum(part, red);
    if (tid == 0) {
      const double x0 = v[j];
      const double nrm = sqrt(nrm2);
      const double alpha = x0 >= 0 ? -nrm : nrm;
      const double v0 = x0 - alpha;
      const double vn2 = __builtin_fma(v0, v0, __builtin_fma(-x0, x0, nrm2));
      s_tau = vn2 > 0 ? 2.0 / vn2 : 0.0;
      aux[j] = s_tau;
      aux[kG + j] = nrm2 > 0 ? alpha : 0.0;
      v[j] = v0;
    }
    __syncthreads();
    const double tau = s_tau;
    if (grp > j) reflect<RK>(v, x[0], j, tau, l);
    if (grp + kGroups > j && grp + kGroups < nG) reflect<RK>(v, x[1], j, tau, l);
    if (grp == j - kGroups * own && l == (j & 15)) {  // the reflector's first element
#pragma unroll
      for (int k = 0; k < RK; ++k)
        if (k == j >> 4) (own ? x[1][k] : x[0][k]) = v[j];
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (grp + kGroups * u < nG) {
#pragma unroll
      for (int k = 0; k < RK; ++k)
        if (l + 16 * k < m) M[(size_t)(grp + kGroups * u) * m + l + 16 * k] = x[u][k];
    }
}

__global__ void __launch_bounds__(kThreads) k_jacobi(int nG, const int* __restrict__ pinv_ptr,
                                                      const double* __restrict__ ws, const double* __restrict__ aux,
                                                      double* __restrict__ Pout) {
  __shared__ double sB[kG * LDB];  // B = R^T, column i at sB[i * LDB]
  __shared__ double sW[kG * LDB];  // rotations, column i at sW[i * LDB]
  __shared__ double sig2[kG];
  __shared__ double s_off[kThreads / 64];
  const int c = blockIdx.x;
  const int off = pinv_ptr[c], m = pinv_ptr[c + 1] - off;
  if (m == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, grp = tid >> 4, l = tid & 15;
  const double* M = ws + (size_t)off * nG;
  const double* rdiag = aux + (size_t)c * kAux + kG;
  double* Z = Pout + (size_t)off * nG;  // column t at Z + t*m (= row t of P_i)
  const int r = min(m, nG);
  // B = R^T (column i of B = row i of R), W = I
  for (int e = tid; e < kG * LDB; e += kThreads) {
    const int i = e / LDB, t = e % LDB;
    double b = 0.0;
    if (i < r && t < nG) b = (t == i) ? rdiag[i] : (t > i ? M[(size_t)t * m + i] : 0.0);
    sB[e] = b;
    sW[e] = (i == t && i < r) ? 1.0 : 0.0;
  }
  __syncthreads();
  // one-sided Jacobi on the r columns of B (round-robin pairs)
  const int np = (r + 1) & ~1;  // players, even
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    double offmax = 0.0;
    // the round's columns of pair grp, 1 + (rd + grp - 1) mod (np - 1) (0 for
    // pair 0) and 1 + (rd + np - 2 - grp) mod (np - 1), stepped
    int ca = (grp - 1 + (np - 1)) % (np - 1), cb = grp < np / 2 ? (np - 2 - grp + (np - 1)) % (np - 1) : 0;
    for (int rd = 0; rd < np - 1; ++rd) {
      // pair grp of the round: lane l holds the elements l + 16k (k < 4) and,
      // l < 2, 64 + l of both columns (entries past nG or r are zero)
      const int a = grp == 0 ? 0 : 1 + ca, b = 1 + cb;
      ca = ca + 1 == np - 1 ? 0 : ca + 1;
      cb = cb + 1 == np - 1 ? 0 : cb + 1;
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
        // the test and the rotation side by side (their chains of square
        // roots and quotients are most of the round)
        const double rel = fabs(ga) / sqrt(al * be);
        const double zeta = (be - al) / (2.0 * ga);
        const double tt = (zeta >= 0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(__builtin_fma(zeta, zeta, 1.0)));
        const double cs = 1.0 / sqrt(__builtin_fma(tt, tt, 1.0)), sn = cs * tt;
        const bool some = !(ga == 0.0 || al == 0.0 || be == 0.0);
        if (some) offmax = fmax(offmax, rel);
        if (some && !(rel < 1e-16)) {
#pragma unroll
          for (int k = 0; k < 5; ++k)
            if (k < 4 || l < kG - 64) {
              const double u = Wa[16 * k], v = Wb[16 * k];
              Ba[16 * k] = __builtin_fma(cs, x[k], -(sn * y[k]));
              Bb[16 * k] = __builtin_fma(sn, x[k], cs * y[k]);
              Wa[16 * k] = __builtin_fma(cs, u, -(sn * v));
              Wb[16 * k] = __builtin_fma(sn, u, cs * v);
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
  // squared singular values, cut-off
  for (int i = w; i < r; i += kThreads / 64) {
    double s = 0.0;
    for (int t = lane; t < nG; t += 64) s = __builtin_fma(sB[i * LDB + t], sB[i * LDB + t], s);
    s = wsum(s);
    if (lane == 0) sig2[i] = s;
  }
  __syncthreads();
  double smax = 0.0;
  for (int i = 0; i < r; ++i) smax = fmax(smax, sig2[i]);
  // X = pinv(R)^T (r x nG): X[k][t] = sum_i W[k][i] B[t][i] / sig2[i] -> Z rows k < r
  for (int e = tid; e < nG * r; e += kThreads) {
    const int k = e % r, t = e / r;
    double x = 0.0;
    for (int i = 0; i < r; ++i)
      if (sig2[i] > kCut * kCut * smax) x += sW[i * LDB + k] * sB[i * LDB + t] / sig2[i];
    Z[(size_t)t * m + k] = x;
  }
}

template <int RK>
__global__ void __launch_bounds__(kThreads) k_apply(int nG, const int* __restrict__ pinv_ptr,
                                                    const double* __restrict__ ws, const double* __restrict__ aux,
                                                    double* __restrict__ Pout) {
  __shared__ double sV[2][16 * RK];
  const int c = blockIdx.x;
  const int off = pinv_ptr[c], m = pinv_ptr[c + 1] - off;
  if (m == 0) return;
  const int tid = threadIdx.x, grp = tid >> 4, l = tid & 15;
  const int r = min(m, nG);
  const double* M = ws + (size_t)off * nG;
  const double* taus = aux + (size_t)c * kAux;
  double* Z = Pout + (size_t)off * nG;
  double x[2][RK];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int k = 0; k < RK; ++k)
      x[u][k] = l + 16 * k < r && grp + kGroups * u < nG ? Z[(size_t)(grp + kGroups * u) * m + l + 16 * k] : 0.0;
  // Z = H_0 ... H_{r-1} Z, the next reflector loaded while one is applied
  auto fetch = [&](int j, int i) { return j >= 0 && i >= j && i < m ? M[(size_t)j * m + i] : 0.0; };
  for (int i = tid; i < 16 * RK; i += kThreads) sV[(r - 1) & 1][i] = fetch(r - 1, i);
  __syncthreads();
  for (int j = r - 1; j >= 0; --j) {
    const double next = fetch(j - 1, tid), tau = taus[j];
    const double more = 16 * RK > kThreads ? fetch(j - 1, tid + kThreads) : 0.0;
    if (grp < nG) reflect<RK>(sV[j & 1], x[0], j, tau, l);
    if (grp + kGroups < nG) reflect<RK>(sV[j & 1], x[1], j, tau, l);
    if (tid < 16 * RK) sV[(j + 1) & 1][tid] = next;
    if (16 * RK > kThreads && tid + kThreads < 16 * RK) sV[(j + 1) & 1][tid + kThreads] = more;
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (grp + kGroups * u < nG) {
#pragma unroll
      for (int k = 0; k < RK; ++k)
        if (l + 16 * k < m) Z[(size_t)(grp + kGroups * u) * m + l + 16 * k] = x[u][k];
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
  if (!D.fac_ws) VFX_HIP(hipMalloc((void**)&D.fac_ws, sizeof(double) * (nv + (size_t)H.ncut * kAux)));
  double* aux = D.fac_ws + nv;
  int most = 0;  // interior points of a cut leaf
  for (int c = 0; c < H.ncut; ++c) most = std::max(most, H.pinv_ptr[c + 1] - H.pinv_ptr[c]);
  const dim3 grid(H.ncut);
  // rows held per lane: 18 cover the paper's grid (K = 8), 30 K = 16 with
  // Kbar = 12, 41 every stencil (there the columns spill)
  static_assert(16 * 41 >= kMaxX, "k_qr holds whole columns");
#define VFX_QR(RKV)                                                                                                 \
  hipLaunchKernelGGL(k_qr<RKV>, grid, dim3(kThreads), 0, s, T.nG, D.pinv_ptr, D.pinv_idx, p->ctx->D.A, D.fac_ws, aux)
#define VFX_APPLY(RKV) \
  hipLaunchKernelGGL(k_apply<RKV>, grid, dim3(kThreads), 0, s, T.nG, D.pinv_ptr, D.fac_ws, aux, D.pinv_val)
  if (most <= 16 * 18)
    VFX_QR(18);
  else if (most <= 16 * 30)
    VFX_QR(30);
  else
    VFX_QR(41);
  hipLaunchKernelGGL(k_jacobi, grid, dim3(kThreads), 0, s, T.nG, D.pinv_ptr, D.fac_ws, aux, D.pinv_val);
  if (most <= 16 * 18)
    VFX_APPLY(18);
  else if (most <= 16 * 30)
    VFX_APPLY(30);
  else
    VFX_APPLY(41);
#undef VFX_QR
#undef VFX_APPLY
  VFX_HIP(hipGetLastError());
  D.factored = true;
  return VFX_OK;
}

}  // namespace vfx
