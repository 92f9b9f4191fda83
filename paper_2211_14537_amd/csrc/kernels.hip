// Device side of the extension + volume FMM path (gfx950, FP64).
//
// Execution order (every output element has one writer, so no atomics are
// needed and results are bitwise reproducible); on the caller's stream, with
// P2L, the near field and M2P on a second one for all but small trees:
//   extension    f^e = f on regular leaves, 0 on leaves outside every
//                extension list, and per cut leaf: f_G = P_i f_{X^I}; values on the Kbar grid of
//                Sbar (given data where interior); total-order Chebyshev
//                expansion; evaluation on every leaf of its extension list
//                (Sections 3.2 and 4.1)
//   moments      exterior moments and multipoles of the leaves (near_sym.hip)
//   up           multipoles of the other boxes
//   p2l, near    list 4 and list 1 from the moments (near_sym.hip), or list 1
//                in mixed precision (mixed.hip, mixed8.hip)
//   m2l          local expansions from list 2 and the list-4 products
//   m2p          list 3
//   down         full local expansions of the leaves
//   far          L2P of the local expansion and the sums of lists 1 and 3
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <mutex>
#include <string>

#include "vfx_internal.h"

namespace vfx {

#define VFX_HIP(call)                                                          \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) {                                                    \
      err = std::string(#call) + ": " + hipGetErrorString(e_);                 \
      return VFX_EHIP;                                                         \
    }                                                                          \
  } while (0)

constexpr int kMaxX = 648;   // |X| for K, Kbar <= 16, deg <= 15
constexpr int kMaxG = 136;
constexpr int kMaxK = 16;
constexpr int kMaxKb = 16;
constexpr double kInv2Pi = 0.15915494309189533576888376337251436;
constexpr double kLn2 = 0.69314718055994530941723212145817657;

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double box_side(double root, int level) { return ldexp(root, -level); }

// -------------------------------------------------------------------------
// Extension of one cut leaf per work-group (NT threads): f_G = P_i f_I
// (A1), values on the Kbar x Kbar grid of Sbar (given data at interior
// nodes, A_{Xbar,G} f_G elsewhere; A2), the total-order Chebyshev
// coefficients (A3) and their values on the K x K nodes of every target
// leaf.  Every global load whose address is known early is issued at the
// start (two waves: indices/geometry, then the data they point to), so the
// work-group's critical path holds few memory round trips.  The time of one
// work-group is the time of the phase on small trees: with at most one cut
// leaf per CU it has 1024 threads (A1 in one pass, four targets at a time);
// more cut leaves run at 256, six work-groups per CU, where the HBM stream of
// the operators becomes the bound.  The phase in us at 256, 512 and 1024
// threads, K = 16 (K = 8): 156 cut leaves 22.8, 20.9, 17.0 (16.9, 14.1, 12.2);
// 196: 24.6, 22.6, 19.0 (19.1, 17.2, 15.1); 308: 27.0, 28.7, 27.7 (20.9, 21.3,
// 22.5); 386: 28.1, 29.1, 28.7 (21.8, 22.4, 23.9); 612: 34.9, 44.0, 40.0 (25.2,
// 35.5, 32.5).
constexpr int kExtTgtMax = 16;  // targets whose geometry is staged in LDS
constexpr int kExtOnePerCu = 256;

// f^e of the leaves no extension list writes, 16-byte pieces e0, e0 +
// step, ... below e1 (piece e: right-hand side e / half, element 2 (e mod
// half)): f on regular leaves (fe_src 1), zero elsewhere (fe_src 0); list
// targets (fe_src 2) are left to their cut leaf's work-group, so every
// element has one writer.
__device__ __forceinline__ void fe_init_range(long e0, long e1, long step, int n, long half,
                                              const int8_t* __restrict__ fe_src, const double* __restrict__ f_leaf,
                                              double* __restrict__ fe, long sfe) {
  // four pieces per round, so their loads are in flight together
  for (long e = e0; e < e1; e += 4 * step) {
    long off[4];
    int src[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long ek = e + k * step;
      const long r = ek / half, i = 2 * (ek - r * half);
      off[k] = r * sfe + i;
      src[k] = ek < e1 ? fe_src[i / n] : 2;
    }
    double2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = src[k] == 1 ? *(const double2*)(f_leaf + off[k]) : make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (src[k] != 2) *(double2*)(fe + off[k]) = v[k];
  }
}

// KT, KBT: compile-time K and Kbar (0: as passed): the index divisions of the
// evaluation by run-time sizes cost a 64-leaf tree 2 us of 45, 4207 leaves
// 4 us of 139
template <int NT, int KT, int KBT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 256 ? 6 : 4))) k_extension(
    int K_, int Kb_, int nX, int nG, const int* __restrict__ pinv_ptr, const uint16_t* __restrict__ pinv_idx,
    const double* __restrict__ pinv_val, const uint8_t* __restrict__ sbar_given, const int* __restrict__ ext_ptr,
    const int* __restrict__ ext_tgt, const double* __restrict__ ext_geo, const double* __restrict__ t,
    const double* __restrict__ AbarT, const double* __restrict__ cbar, const double* __restrict__ f_cut,
    double* __restrict__ fe, int nrhs, long sfc, long sfe, int ext_blocks, int L,
    const int8_t* __restrict__ fe_src, const double* __restrict__ f_leaf) {
  const int K = KT ? KT : K_, Kb = KBT ? KBT : Kb_;
  const long half = (long)L * K * K / 2, pieces = half * nrhs;
  if ((int)blockIdx.x >= ext_blocks) {
    // the work-groups past the cut leaves initialise f^e of the other
    // leaves, grid-stride (they take the slots the cut leaves free)
    const long nb = (long)(gridDim.x - ext_blocks) * blockDim.x;
    fe_init_range((long)(blockIdx.x - ext_blocks) * blockDim.x + threadIdx.x, pieces, nb, K * K, half, fe_src,
                  f_leaf, fe, sfe);
    return;
  }
  // consecutive work-groups take the right-hand sides of one cut leaf, so
  // its operator P_i is read from HBM once and reused from L2
  const int rhs = blockIdx.x % nrhs;
  f_cut += rhs * sfc;
  fe += rhs * sfe;
  __shared__ double s_fI[kMaxX];
  __shared__ double s_fG[kMaxG];
  __shared__ double s_cb[kMaxKb * kMaxKb];
  __shared__ double s_g[kMaxKb * kMaxKb];
  __shared__ double s_coef[kMaxKb * kMaxKb];
  // targets evaluated side by side, 256 threads each
  constexpr int TQ = NT / 256, TB = kMaxK * kMaxKb;
  __shared__ double s_tmpq[TQ * TB], s_Exq[TQ * TB], s_Eyq[TQ * TB];
  double* const s_tmp = s_tmpq;
  __shared__ double s_t[kMaxK];
  __shared__ double s_geo[3 * kExtTgtMax];
  __shared__ int s_tg[kExtTgtMax];
  __shared__ uint8_t s_given[kMaxKb * kMaxKb];
  const int c = blockIdx.x / nrhs;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: row indices in scalar registers
  const int n = K * K, Kb2 = Kb * Kb;
  const int off = pinv_ptr[c], ni = pinv_ptr[c + 1] - off;
  const int e0 = ext_ptr[c], ne = ext_ptr[c + 1] - e0;
  const double* fc = f_cut + (size_t)c * nX;
  // A2's operator does not wait for anything: with threads to spare, thread
  // (a, hf) takes the even (hf = 0) or odd rows of one Sbar point into
  // registers now (the default stencil of 66 support nodes)
  const bool early = NT > 256 && nG == 66;
  const int hf = tid / Kb2, ga = tid - hf * Kb2;
  double wA[NT > 256 ? 34 : 1];
  if constexpr (NT > 256) {
    if (early && hf < 2) {
#pragma unroll
      for (int u = 0; u < 32; ++u) wA[u] = AbarT[(size_t)(2 * u + hf) * Kb2 + ga];
      wA[32] = AbarT[(size_t)64 * Kb2 + ga];
      wA[33] = AbarT[(size_t)65 * Kb2 + ga];
    }
  }
  // first load wave: indices, flags, small tables, target geometry
  int idx0 = tid < ni ? pinv_idx[off + tid] : 0;
  int idx1 = tid + NT < ni ? pinv_idx[off + tid + NT] : 0;
  const bool given = tid < Kb2 && sbar_given[(size_t)c * Kb2 + tid];
  if (tid < Kb2) s_cb[tid] = cbar[tid];
  if (tid < K) s_t[tid] = t[tid];
  if (tid < ne && tid < kExtTgtMax) {
    s_tg[tid] = ext_tgt[e0 + tid];
    s_geo[3 * tid] = ext_geo[3 * (e0 + tid)];
    s_geo[3 * tid + 1] = ext_geo[3 * (e0 + tid) + 1];
    s_geo[3 * tid + 2] = ext_geo[3 * (e0 + tid) + 2];
  }
  // second load wave: interior samples and the given Sbar-grid values
  if (tid < ni) s_fI[tid] = fc[idx0];
  if (tid + NT < ni) s_fI[tid + NT] = fc[idx1];
  for (int q = tid + 2 * NT; q < ni; q += NT) s_fI[q] = fc[pinv_idx[off + q]];
  if (tid < Kb2) {
    s_given[tid] = given;
    if (given) s_g[tid] = fc[n + tid];
  }
  __syncthreads();
  // A1: f_G = P_i f_I  (P_i: nG x ni row-major).  Wave w takes 4096 / NT rows
  // in passes of 4, lane l the columns l, l + 64, l + 128,
  // l + 192 (then l + 256, ... for ni > 256): one pass reads four whole rows
  // (ni <= 256), every load of a wave 512 contiguous bytes, 16 loads in
  // flight at once.  The 4 row partials are combined across the lanes by a
  // recursive-halving reduce-scatter over lane bits 1..0 (lane l ends with
  // row l & 3) and four plain butterfly steps over bits 2..5.  Rows >= 64
  // (a stencil degree above 10) use wave sums.  Few live registers keep six
  // work-groups per CU resident, so the operators of all cut leaves stream
  // at once; P_i is read once per execute, so its loads are non-temporal
  // (they do not displace the data the later kernels reuse).
  const double* P = pinv_val + (size_t)off * nG;
#pragma unroll 1
  for (int pass = 0; pass < 1024 / NT; ++pass) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int r0 = 4096 / NT * wave + 4 * pass;
#pragma unroll 1
    for (int q = lane; q < ni; q += 256) {
      double f[4], p[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = q + 64 * j < ni ? s_fI[q + 64 * j] : 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = min(r0 + r, nG - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          p[r][j] = q + 64 * j < ni ? __builtin_nontemporal_load(P + row * ni + q + 64 * j) : 0.0;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double m = (r0 + r < nG) ? 1.0 : 0.0;
        acc[r] += m * (p[r][0] * f[0] + p[r][1] * f[1] + p[r][2] * f[2] + p[r][3] * f[3]);
      }
    }
#pragma unroll
    for (int s = 2; s >= 1; s >>= 1) {
      const bool up = (lane & s) != 0;
#pragma unroll
      for (int j = 0; j < s; ++j) {
        const double send = up ? acc[j] : acc[j + s];
        const double keep = up ? acc[j + s] : acc[j];
        acc[j] = keep + __shfl_xor(send, s, 64);
      }
    }
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) acc[0] += __shfl_xor(acc[0], o, 64);
    if (lane < 4 && r0 + lane < nG) s_fG[r0 + lane] = acc[0];
  }
  for (int r = 64 + wave; r < nG; r += NT / 64) {
    double a = 0.0;
    const double* pr = P + (size_t)r * ni;
    for (int q = lane; q < ni; q += 64) a += pr[q] * s_fI[q];
    a = wave_sum(a);
    if (lane == 0) s_fG[r] = a;
  }
  __syncthreads();
  // A2: the Sbar grid values not given as data, A_{Xbar,G} f_G (universal
  // operator rows in batches of 16 independent loads)
  if constexpr (NT > 256) {
    if (early) {
      if (hf < 2) {  // the sums of the general path below, its two halves apart
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < 32; ++u) v = __builtin_fma(wA[u], s_fG[2 * u + hf], v);
        if (hf == 0) {
          v = __builtin_fma(wA[32], s_fG[64], v);
          v = __builtin_fma(wA[33], s_fG[65], v);
        }
        s_tmp[tid] = v;
      }
      __syncthreads();
      if (tid < Kb2 && !s_given[tid]) s_g[tid] = s_tmp[tid] + s_tmp[Kb2 + tid];
    }
  }
  for (int a = tid; a < Kb2 && !early; a += NT) {
    if (s_given[a]) continue;
    double v0 = 0.0, v1 = 0.0;
    int r = 0;
    for (; r + 16 <= nG; r += 16) {
      double w[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) w[u] = AbarT[(size_t)(r + u) * Kb2 + a];
#pragma unroll
      for (int u = 0; u < 16; u += 2) {
        v0 += w[u] * s_fG[r + u];
        v1 += w[u + 1] * s_fG[r + u + 1];
      }
    }
    for (; r < nG; ++r) v0 += AbarT[(size_t)r * Kb2 + a] * s_fG[r];
    s_g[a] = v0 + v1;
  }
  __syncthreads();
  // A3: coefficients c = C g C^T, truncated to total order < Kbar
  for (int e = tid; e < Kb2; e += NT) {
    const int m = e / Kb, j = e % Kb;
    double acc = 0.0;
    for (int i = 0; i < Kb; ++i) acc += s_cb[m * Kb + i] * s_g[i * Kb + j];
    s_tmp[e] = acc;
  }
  __syncthreads();
  for (int e = tid; e < Kb2; e += NT) {
    const int m = e / Kb, nn = e % Kb;
    double acc = 0.0;
    if (m + nn < Kb)
      for (int j = 0; j < Kb; ++j) acc += s_tmp[m * Kb + j] * s_cb[nn * Kb + j];
    s_coef[e] = acc;
  }
  __syncthreads();
  // values at the K x K nodes of every target leaf (the cut leaf first), TQ
  // targets at a time
  const int sub = wave / 4, st = tid & 255;
  double *tq = s_tmpq + sub * TB, *Ex = s_Exq + sub * TB, *Ey = s_Eyq + sub * TB;
  for (int q0 = 0; q0 < ne; q0 += TQ) {
    const int q = q0 + sub;
    int j = 0;
    double ox = 0.0, oy = 0.0, sc = 0.0;
    if (q < ne) {
      if (q < kExtTgtMax) {
        j = s_tg[q];
        ox = s_geo[3 * q];
        oy = s_geo[3 * q + 1];
        sc = s_geo[3 * q + 2];
      } else {
        j = ext_tgt[e0 + q];
        ox = ext_geo[3 * (e0 + q)];
        oy = ext_geo[3 * (e0 + q) + 1];
        sc = ext_geo[3 * (e0 + q) + 2];
      }
    }
    if (st < 2 * K) {
      const int a = st % K;
      const bool isy = st >= K;
      const double xi = (isy ? oy : ox) + sc * s_t[a];
      double* dst = (isy ? Ey : Ex) + a * Kb;
      double t0 = 1.0, t1 = xi;
      dst[0] = 1.0;
      if (Kb > 1) dst[1] = xi;
      for (int m = 2; m < Kb; ++m) {
        const double t2 = 2.0 * xi * t1 - t0;
        dst[m] = t2;
        t0 = t1;
        t1 = t2;
      }
    }
    __syncthreads();
    for (int idx = st; idx < Kb * K; idx += 256) {
      const int m = idx / K, b = idx % K;
      double acc = 0.0;
      for (int nn = 0; nn < Kb - m; ++nn) acc += s_coef[m * Kb + nn] * Ey[b * Kb + nn];
      tq[idx] = acc;
    }
    __syncthreads();
    if (q < ne)
      for (int idx = st; idx < n; idx += 256) {
        const int a = idx / K, b = idx % K;
        double acc = 0.0;
        for (int m = 0; m < Kb; ++m) acc += Ex[a * Kb + m] * tq[m * K + b];
        fe[(size_t)j * n + idx] = acc;
      }
    __syncthreads();
  }
}

typedef double vfx_d4 __attribute__((ext_vector_type(4)));
typedef double vfx_d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// calls f(integral_constant<int, I>) for I = I0 .. N-1 (ring indices in an
// unrolled pipeline stay compile-time constants)
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Per-output rows of the lane-per-pair kernels' LDS staging: 65 (not 64)
// double2 apart, so the eight lanes of a segment that read the same entry
// of eight outputs fall in different banks.
constexpr int kSoStride = 65;

// Sum of s[q] over q in [q0, q1) in a fixed order with four
// interleaved partial sums (deterministic, and the LDS loads overlap).
__device__ __forceinline__ double2 seg_sum(const double2* s, int q0, int q1) {
  double r0 = 0.0, i0 = 0.0, r1 = 0.0, i1 = 0.0, r2 = 0.0, i2 = 0.0, r3 = 0.0, i3 = 0.0;
  int q = q0;
  for (; q + 3 < q1; q += 4) {
    const double2 v0 = s[q], v1 = s[q + 1], v2 = s[q + 2], v3 = s[q + 3];
    r0 += v0.x;
    i0 += v0.y;
    r1 += v1.x;
    i1 += v1.y;
    r2 += v2.x;
    i2 += v2.y;
    r3 += v3.x;
    i3 += v3.y;
  }
  for (; q < q1; ++q) {
    r0 += s[q].x;
    i0 += s[q].y;
  }
  return make_double2((r0 + r1) + (r2 + r3), (i0 + i1) + (i2 + i3));
}

// M2L with one lane per list-2 entry (target box, source box), for a group
// of consecutive target boxes with at most 64 entries and at most 8 boxes.
// Lane e holds s_k = (-t)^k a_k of its source (registers); the shared
// Pascal coefficients C(k+l-1,l) are wave-uniform operands.  For each output
// l the lane forms t^l sum_k C(k+l-1,l) s_k (minus a_0 t^l/l, plus the log
// term for l = 0); the per-target sums go through LDS in chunks of 8 outputs,
// in entry order (deterministic), together with the P2L contributions.
template <int PM>
__global__ void __launch_bounds__(64) k_m2l_pairs(int P, double root_size, const int* __restrict__ grp,
                                                  const int* __restrict__ box_level, const int* __restrict__ l2_ptr,
                                                  const int* __restrict__ l2_src, const int* __restrict__ l2_off,
                                                  const int* __restrict__ l2_tgt, const int* __restrict__ l4_ptr,
                                                  const int* __restrict__ l4_src, const int* __restrict__ l4_slot,
                                                  const int* __restrict__ leaf_box, int p2l_rows,
                                                  const double* __restrict__ pasT, const double* __restrict__ logd,
                                                  const double2* __restrict__ mpole, const double* __restrict__ p2l_y,
                                                  double2* __restrict__ local, long smp, long spl) {
  mpole += blockIdx.y * smp;  // right-hand side blockIdx.y
  local += blockIdx.y * smp;
  p2l_y += blockIdx.y * spl;
  __shared__ double2 s_o[8 * kSoStride];
  const int g = blockIdx.x;
  const int b0 = grp[g], b1 = grp[g + 1];
  const int e0 = l2_ptr[b0], e1 = l2_ptr[b1];
  const int lane = threadIdx.x;
  const int e = e0 + lane;
  const bool act = e < e1;
  const int o = act ? l2_off[e] : 0;
  const int src = act ? l2_src[e] : 0;
  const double dx = (o / 7) - 3, dy = (o % 7) - 3;
  const double dd = (dx * dx + dy * dy) > 0 ? dx * dx + dy * dy : 1.0;
  const double2 t = make_double2(dx / dd, -dy / dd);  // 1 / (dx + i dy)
  double2 s[PM];
  {
    double2 pw = make_double2(1.0, 0.0);
    const double2 mt = make_double2(-t.x, -t.y);
#pragma unroll
    for (int k = 0; k < PM; ++k) {
      const double2 a = (act && k < P) ? mpole[(size_t)src * P + k] : make_double2(0.0, 0.0);
      s[k] = cmul(pw, a);
      pw = cmul(pw, mt);
    }
  }
  const double a0 = s[0].x;
  const int tgt = act ? l2_tgt[e] : b0;
  const double logh = log(box_side(root_size, box_level[tgt]));
  const double lg0 = act ? a0 * (logd[o] + logh) : 0.0;
  double2 tl = make_double2(1.0, 0.0);
  const int nchunk = (P + 7) / 8;
  for (int c = 0; c < nchunk; ++c) {
    double2 outc[8];
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) {
      const int l = 8 * c + lc;
      double2 out = make_double2(0.0, 0.0);
      if (l < P) {
        const double* cr = pasT + (size_t)l * P;
        double ur = 0.0, ui = 0.0;
#pragma unroll
        for (int k = 1; k < PM; ++k) {
          if (k < P) {
            const double cf = cr[k];
            ur += cf * s[k].x;
            ui += cf * s[k].y;
          }
        }
        out = cmul(tl, make_double2(ur, ui));
        if (l == 0) {
          out.x += lg0;
        } else {
          out.x -= a0 * tl.x / l;
          out.y -= a0 * tl.y / l;
        }
        tl = cmul(tl, t);
      }
      outc[lc] = act ? out : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) s_o[lc * kSoStride + lane] = outc[lc];
    __syncthreads();
    const int lc = lane & 7, seg = lane >> 3;
    const int bb = b0 + seg, l = 8 * c + lc;
    if (bb < b1 && l < P) {
      const double2 sv = seg_sum(s_o + lc * kSoStride, l2_ptr[bb] - e0, l2_ptr[bb + 1] - e0);
      double re = sv.x, im = sv.y;
      const double h = box_side(root_size, box_level[bb]);
      const double h2 = h * h;
      for (int q = l4_ptr[bb]; q < l4_ptr[bb + 1]; ++q) {
        const double* y = p2l_y + (size_t)l4_slot[q] * p2l_rows + 2 * l;
        re += h2 * y[0];
        im += h2 * y[1];
        if (l == 0) re += log(h) * mpole[(size_t)leaf_box[l4_src[q]] * P].x;
      }
      local[(size_t)bb * P + l] = make_double2(re, im);
    }
  }
}

// -------------------------------------------------------------------------
// Lane-per-translation forms, instantiated for the exact expansion length P
// (compile-time loops, so the Pascal coefficients, read through wave-uniform
// pointers, become scalar operands of the FMAs and need no LDS traffic).

// complex product with its fused operations named: both forms of k_m2l_lanes
// round alike, so a right-hand side of a batch keeps the bits of a single
// execute whichever form each takes
__device__ __forceinline__ double2 cmul_fma(double2 a, double2 b) {
  return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}

// M2L: one lane per list-2 entry (target, source), for a group of
// consecutive target boxes with at most 64 entries and at most 8 boxes.
// Lane e holds s_k = (-t)^k a_k of its source; for each output l it forms
// t^l sum_k C(k+l-1,l) s_k (minus a_0 t^l/l; plus a_0 (log|d/h| + log h) for
// l = 0).  Per-target sums go through LDS in chunks of 8 outputs, in entry
// order (deterministic), together with the P2L contributions.  SPLIT (small
// trees, whose groups leave SIMDs empty): one work-group per chunk of outputs,
// each forming the s_k again.
template <int P, bool SPLIT>
__global__ void __launch_bounds__(64) k_m2l_lanes(double root_size, const int* __restrict__ grp,
                                                  const int* __restrict__ box_level, const int* __restrict__ l2_ptr,
                                                  const int* __restrict__ l2_src, const int* __restrict__ l2_off,
                                                  const int* __restrict__ l2_tgt, const int* __restrict__ l4_ptr,
                                                  const int* __restrict__ l4_src, const int* __restrict__ l4_slot,
                                                  const int* __restrict__ leaf_box, int p2l_rows,
                                                  const double* __restrict__ pasT, const double* __restrict__ logd,
                                                  const double2* __restrict__ mpole, const double* __restrict__ p2l_y,
                                                  double2* __restrict__ local, long smp, long spl) {
  mpole += blockIdx.y * smp;  // right-hand side blockIdx.y
  local += blockIdx.y * smp;
  p2l_y += blockIdx.y * spl;
  __shared__ double2 s_o[8 * kSoStride];
  const int g = blockIdx.x;
  const int b0 = grp[g], b1 = grp[g + 1];
  const int e0 = l2_ptr[b0], e1 = l2_ptr[b1];
  const int lane = threadIdx.x;
  const int e = e0 + lane;
  const bool act = e < e1;
  const int o = act ? l2_off[e] : 0;
  const int src = act ? l2_src[e] : 0;
  const double dx = (o / 7) - 3, dy = (o % 7) - 3;
  const double dd = dx * dx + dy * dy;
  const double2 t = make_double2(dx / dd, -dy / dd);  // 1 / (dx + i dy)
  double2 s[P];
  {
    double2 pw = make_double2(1.0, 0.0);
    const double2 mt = make_double2(-t.x, -t.y);
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const double2 a = act ? mpole[(size_t)src * P + k] : make_double2(0.0, 0.0);
      s[k] = cmul_fma(pw, a);
      pw = cmul_fma(pw, mt);
    }
  }
  const double a0 = s[0].x;
  const int tgt = act ? l2_tgt[e] : b0;
  const double lg0 = act ? a0 * (logd[o] + log(box_side(root_size, box_level[tgt]))) : 0.0;
  double2 tl = make_double2(1.0, 0.0);
  constexpr int NC = (P + 7) / 8;
  // this lane's output role in every chunk: box bb = b0 + seg, outputs
  // l = 8c + lc; its list-2 range and the P2L contributions (h^2 times the
  // list-4 products, and log(h) a_0 of each list-4 leaf for l = 0) are
  // gathered once, here, so the chunk tails only sum LDS and store
  const int lc = lane & 7, seg = lane >> 3;
  const int bb = b0 + seg;
  const bool own = bb < b1;
  int r0 = 0, r1 = 0;
  constexpr int NP = SPLIT ? 1 : NC;  // chunks this work-group forms
  const int c0 = SPLIT ? (int)blockIdx.z : 0;
  double p2r[NP], p2i[NP];
#pragma unroll
  for (int c = 0; c < NP; ++c) p2r[c] = p2i[c] = 0.0;
  if (own) {
    r0 = l2_ptr[bb] - e0;
    r1 = l2_ptr[bb + 1] - e0;
    const double h = box_side(root_size, box_level[bb]);
    const double h2 = h * h;
    const int q0 = l4_ptr[bb], q1 = l4_ptr[bb + 1];
    double lgs = 0.0;
    for (int q = q0; q < q1; ++q) {
      const double* y = p2l_y + (size_t)l4_slot[q] * p2l_rows + 2 * lc;
#pragma unroll
      for (int c = 0; c < NP; ++c)
        if (8 * (c0 + c) + lc < P) {
          p2r[c] = __builtin_fma(h2, y[16 * (c0 + c)], p2r[c]);
          p2i[c] = __builtin_fma(h2, y[16 * (c0 + c) + 1], p2i[c]);
        }
      if (lc == 0) lgs += mpole[(size_t)leaf_box[l4_src[q]] * P].x;
    }
    if (c0 == 0) p2r[0] = __builtin_fma(log(h), lgs, p2r[0]);  // zero unless lc == 0 (output l = 0)
  }
  static_for<0, NC>([&](auto cc) __attribute__((always_inline)) {
    constexpr int c = decltype(cc)::value;
    if (SPLIT && c != c0) {
      if (c < c0) {  // on to t^(8c), the same product sequence as below
#pragma unroll
        for (int i = 0; i < 8; ++i) tl = cmul_fma(tl, t);
      }
      return;
    }
    __syncthreads();
    // the eight outputs of the chunk accumulate side by side (k outer), so
    // their FMA chains interleave
    double ur[8], ui[8];
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) ur[lc] = ui[lc] = 0.0;
#pragma unroll
    for (int k = 1; k < P; ++k) {
#pragma unroll
      for (int lc = 0; lc < 8; ++lc) {
        const int l = 8 * c + lc;
        if (l < P) {
          const double cf = pasT[l * P + k];
          ur[lc] = __builtin_fma(cf, s[k].x, ur[lc]);
          ui[lc] = __builtin_fma(cf, s[k].y, ui[lc]);
        }
      }
    }
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) {
      const int l = 8 * c + lc;
      double2 out = make_double2(0.0, 0.0);
      if (l < P) {
        out = cmul_fma(tl, make_double2(ur[lc], ui[lc]));
        if (l == 0) {
          out.x += lg0;
        } else {
          const double il = 1.0 / (double)l;  // compile-time constant
          out.x = __builtin_fma(-(a0 * tl.x), il, out.x);
          out.y = __builtin_fma(-(a0 * tl.y), il, out.y);
        }
        tl = cmul_fma(tl, t);
      }
      s_o[lc * kSoStride + lane] = act ? out : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int l = 8 * c + lc;
    if (own && l < P) {
      const double2 sv = seg_sum(s_o + lc * kSoStride, r0, r1);
      local[(size_t)bb * P + l] = make_double2(sv.x + p2r[SPLIT ? 0 : c], sv.y + p2i[SPLIT ? 0 : c]);
    }
  });
}

// -------------------------------------------------------------------------
// Batched table GEMMs on the FP64 matrix cores (M2P, the factor products of
// the target-stationary near field): entries (pairs) are grouped by table
// configuration c, and every entry e of a tile gets
//   Y[e][row] = sum_k A_c[k][row] X[src(e)][k].
//   A: [c][k][row], R = 16*MT rows (rows fastest, MT a multiple of MTB);
//   X: [src][k] with row stride ldx, values k >= kx taken as zero (M2P reads
//   the 2P coefficients of a multipole); Y: [e][row].
// v_mfma_f64_16x16x4f64: lane l holds A[l%16][l/16], B[l/16][l%16] and the
// outputs D[(l/16) + 4r][l%16], r = 0..3 (lane layout checked on gfx950).
// A work item is a tile of <= 64 entries of one configuration and a block of
// MTB row tiles; wave w owns the entries 16w..16w+15.  The entry operands go straight from memory into a ring of
// three register blocks (contraction order permuted so that a lane reads 64
// contiguous bytes per block: MFMA step s of block kb pairs k = 32kb +
// 8(l/16) + s with lane l on both sides); the table block (32 k x 16 MTB
// rows), shared by the four waves, goes through a ring of two register
// blocks into double-buffered LDS.  Every global load is issued two
// compute phases before its data is needed.  LDS rows are 16 MTB + 2
// doubles apart, so the two lane groups of a half-wave (rows 8 apart) fall
// into opposite halves of the banks.  XCD-aware, persistent order:
// work-groups are dispatched round-robin over the 8 XCDs, so those of XCD x
// (blockIdx % 8 == x) walk one contiguous range of work items; consecutive
// items share a configuration and hence a table, which that XCD's L2 then
// serves to all of them.
template <int KD, int MTB>
__global__ void __launch_bounds__(256) k_tgemm(int nitems, int MT, const int* __restrict__ t_cfg,
                                               const int* __restrict__ t_first, const int* __restrict__ t_count,
                                               const int* __restrict__ src, const double* __restrict__ A,
                                               const double* __restrict__ X, double* __restrict__ Y, long sx,
                                               long sy, int ldx, int kx) {
  static_assert(KD % 32 == 0, "contraction in blocks of 32");
  X += blockIdx.y * sx;  // right-hand side blockIdx.y
  Y += blockIdx.y * sy;
  constexpr int KB = 32, NKB = KD / KB;
  constexpr int NC = 16 * MTB, LDB = NC + 2;  // table columns per block, LDS row stride
  constexpr int BP = NC / 2;                  // 16-byte pieces per table row
  __shared__ __attribute__((aligned(16))) double sB[2 * KB * LDB];
  const int nrb = MT / MTB;
  const int nb = gridDim.x, bb = blockIdx.x;
  const int x = bb & 7;
  const int q = nitems >> 3, rr = nitems & 7;
  const int xfirst = x * q + min(x, rr), xcount = q + (x < rr ? 1 : 0);
  const int xwgs = (nb - x + 7) >> 3;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int R = 16 * MT;
  for (int j = bb >> 3; j < xcount; j += xwgs) {
    const int item = xfirst + j;
    const int tile = item / nrb, rb = item - tile * nrb;
    const int c = t_cfg[tile], p0 = t_first[tile], np = t_count[tile];
    const int row0 = NC * rb;
    const double* Ac = A + (size_t)c * KD * R + row0;
    // this lane's entry (an entry past the tile's end reads the first
    // entry's row; its results are not stored)
    const int ent = 16 * w + li;
    const double* xrow = X + (size_t)src[p0 + (ent < np ? ent : 0)] * ldx + 8 * lk;
    vfx_d2 ra[3][4], rbuf[2][MTB];
    auto ga = [&](auto kbc, auto slot) __attribute__((always_inline)) {
      constexpr int kb = decltype(kbc)::value, sl = decltype(slot)::value;
      static_for<0, 4>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        ra[sl][e] =
            (KB * kb + 8 * lk + 2 * e < kx) ? *(const vfx_d2*)(xrow + KB * kb + 2 * e) : vfx_d2{0.0, 0.0};
      });
    };
    auto gb = [&](auto kbc, auto slot) __attribute__((always_inline)) {
      constexpr int kb = decltype(kbc)::value, sl = decltype(slot)::value;
      static_for<0, MTB>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        const int qq = tid + 256 * e, row = qq / BP, col = 2 * (qq % BP);
        rbuf[sl][e] = *(const vfx_d2*)(Ac + (size_t)(KB * kb + row) * R + col);
      });
    };
    auto sb = [&](auto buf, auto slot) __attribute__((always_inline)) {
      constexpr int bf = decltype(buf)::value, sl = decltype(slot)::value;
      static_for<0, MTB>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        const int qq = tid + 256 * e, row = qq / BP, col = 2 * (qq % BP);
        *(vfx_d2*)(sB + (bf * KB + row) * LDB + col) = rbuf[sl][e];
      });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    vfx_d4 acc[MTB];
#pragma unroll
    for (int r = 0; r < MTB; ++r) acc[r] = vfx_d4{0, 0, 0, 0};
    ga(I0{}, I0{});
    gb(I0{}, I0{});
    if constexpr (NKB > 1) {
      ga(I1{}, I1{});
      gb(I1{}, I1{});
    }
    __syncthreads();  // the previous item is done with sB
    sb(I0{}, I0{});
    __syncthreads();
    static_for<0, NKB>([&](auto kbc) __attribute__((always_inline)) {
      constexpr int kb = decltype(kbc)::value;
      if constexpr (kb + 2 < NKB) {
        ga(std::integral_constant<int, kb + 2>{}, std::integral_constant<int, (kb + 2) % 3>{});
        gb(std::integral_constant<int, kb + 2>{}, std::integral_constant<int, kb % 2>{});
      }
      const double* sbk = sB + ((kb % 2) * KB + 8 * lk) * LDB + li;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const double av = (s & 1) ? ra[kb % 3][s >> 1].y : ra[kb % 3][s >> 1].x;
        double bv[MTB];
#pragma unroll
        for (int r = 0; r < MTB; ++r) bv[r] = sbk[s * LDB + 16 * r];
#pragma unroll
        for (int r = 0; r < MTB; ++r) acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[r], acc[r], 0, 0, 0);
      }
      if constexpr (kb + 1 < NKB) sb(std::integral_constant<int, (kb + 1) % 2>{}, std::integral_constant<int, (kb + 1) % 2>{});
      __syncthreads();
    });
    // outputs D[lk + 4e][16 r + li]: entry 16w + lk + 4e, row row0 + 16r + li
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int en = 16 * w + lk + 4 * e;
      if (en >= np) continue;
#pragma unroll
      for (int r = 0; r < MTB; ++r) Y[(size_t)(p0 + en) * R + row0 + 16 * r + li] = acc[r][e];
    }
  }
}

// -------------------------------------------------------------------------
// Upward pass without the level-by-level chain.  The multipole of a non-leaf
// box B (level >= 2) about its own centre is the sum, over the leaves L below
// it, of the leaf multipoles shifted to B.  The shifted coefficients b_l
// depend only on a_k with k <= l, so they are exact (up to rounding) for any
// number of levels between L and B.  Scaled form (a_k h_L^-k, b_l h_B^-l):
//   b_0 = a_0,  b_l = w^l [ sum_{1<=k<=l} C(l-1,k-1) (r/w)^k a_k - a_0/l ],
// w = (c_L - c_B)/h_B, r = h_L/h_B.  One lane per (box, leaf) pair; a group
// of <= 8 boxes and <= 64 pairs per wave; per-box sums in pair order through
// LDS (deterministic).  Slices of a box with more than 64 pairs write
// partial sums, added in slice order by k_up_sum.
template <int PM, bool EXACT>
__global__ void __launch_bounds__(64) k_up(int Prt, double root_size, const int* __restrict__ grp, const int* __restrict__ up_box,
                                           const int* __restrict__ up_ptr, const int* __restrict__ up_src,
                                           const int* __restrict__ up_pos, const int* __restrict__ box_level,
                                           const double* __restrict__ box_cx, const double* __restrict__ box_cy,
                                           const double* __restrict__ pasT, double2* __restrict__ mpole,
                                           double2* __restrict__ part, long smp, long spart) {
  const int P = EXACT ? PM : Prt;
  mpole += blockIdx.y * smp;  // right-hand side blockIdx.y
  part += blockIdx.y * spart;
  __shared__ double2 s_o[8 * kSoStride];
  const int* gg = grp + 5 * blockIdx.x;
  const int u0 = gg[0], u1 = gg[1], e0 = gg[2], e1 = gg[3], slot = gg[4];
  const int lane = threadIdx.x;
  const int e = e0 + lane;
  const bool act = e < e1;
  const int src = act ? up_src[e] : up_box[u0];
  const int tgt = up_box[act ? up_pos[e] : u0];
  const int ls = box_level[src], lt = box_level[tgt];
  const double hb = box_side(root_size, lt);
  const double2 w = act ? make_double2((box_cx[src] - box_cx[tgt]) / hb, (box_cy[src] - box_cy[tgt]) / hb)
                        : make_double2(0.5, 0.5);
  const double r = act ? ldexp(1.0, lt - ls) : 1.0;
  const double ww = w.x * w.x + w.y * w.y;
  const double2 q = make_double2(r * w.x / ww, -r * w.y / ww);  // r / w
  const int NC = (P + 7) / 8;
  // work-group z computes the outputs l = 8c .. 8c+7 (chunk c = blockIdx.z,
  // a compile-time constant inside the matching branch); the scaled source
  // coefficients s_k = (r/w)^k a_k, k <= 8c+7, are formed on the fly (k
  // outer) rather than held, which keeps the kernel at a few dozen registers
  static_for<0, (PM + 7) / 8>([&](auto cc) __attribute__((always_inline)) {
    constexpr int c = decltype(cc)::value;
    constexpr int KH = (8 * c + 8 < PM) ? 8 * c + 8 : PM;  // k < KH
    if (c != (int)blockIdx.z || c >= NC) return;
    // w^(l-1) before output l: the same product sequence as a running power
    double2 wl = make_double2(1.0, 0.0);
#pragma unroll
    for (int i = 1; i < 8 * c; ++i) wl = cmul(wl, w);
    double2 pw = make_double2(1.0, 0.0);
    const double2 a0 = cmul(pw, act ? mpole[(size_t)src * P] : make_double2(0.0, 0.0));
    pw = cmul(pw, q);
    // the eight outputs of the chunk accumulate side by side (k outer)
    double ur[8], ui[8];
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) {
      const int l = 8 * c + lc;
      const double il = l > 0 ? 1.0 / (double)l : 0.0;  // compile-time constant
      ur[lc] = -a0.x * il;
      ui[lc] = -a0.y * il;
    }
#pragma unroll
    for (int k = 1; k < KH; ++k) {
      const double2 a = (act && k < P) ? mpole[(size_t)src * P + k] : make_double2(0.0, 0.0);
      const double2 sk = cmul(pw, a);
      pw = cmul(pw, q);
#pragma unroll
      for (int lc = 0; lc < 8; ++lc) {
        const int l = 8 * c + lc;
        if (k <= l && l < P) {
          const double cf = pasT[l * P + k];
          ur[lc] += cf * sk.x;
          ui[lc] += cf * sk.y;
        }
      }
    }
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) {
      const int l = 8 * c + lc;
      double2 out = make_double2(0.0, 0.0);
      if (l == 0) {
        out = a0;
      } else if (l < P) {
        wl = cmul(wl, w);
        out = cmul(wl, make_double2(ur[lc], ui[lc]));
      }
      s_o[lc * kSoStride + lane] = act ? out : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int lc = lane & 7, seg = lane >> 3;
    const int uu = u0 + seg, l = 8 * c + lc;
    if (uu < u1 && l < P) {
      const int q0 = max(up_ptr[uu], e0), q1 = min(up_ptr[uu + 1], e1);
      const double2 sv = seg_sum(s_o + lc * kSoStride, q0 - e0, q1 - e0);
      const double re = sv.x, im = sv.y;
      if (slot < 0)
        mpole[(size_t)up_box[uu] * P + l] = make_double2(re, im);
      else
        part[(size_t)slot * P + l] = make_double2(re, im);
    }
  });
}

// Multipoles of the split boxes: the slices' partial sums added in a fixed
// order (eight running sums, slice j into sum j mod 8, then combined
// pairwise), eight loads in flight per round rather than one round trip per
// slice.
__global__ void __launch_bounds__(64) k_up_sum(int P, const int* __restrict__ split, const double2* __restrict__ part,
                                               double2* __restrict__ mpole, long spart, long smp) {
  part += blockIdx.y * spart;  // right-hand side blockIdx.y
  mpole += blockIdx.y * smp;
  const int* sp = split + 3 * blockIdx.x;
  const int l = threadIdx.x;
  if (l >= P) return;
  const int first = sp[1], ns = sp[2];
  double re[8], im[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) re[u] = im[u] = 0.0;
  for (int j = 0; j < ns; j += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = j + u < ns ? part[(size_t)(first + j + u) * P + l] : make_double2(0.0, 0.0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      re[u] += v[u].x;
      im[u] += v[u].y;
    }
  }
  const double r = ((re[0] + re[1]) + (re[2] + re[3])) + ((re[4] + re[5]) + (re[6] + re[7]));
  const double i = ((im[0] + im[1]) + (im[2] + im[3])) + ((im[4] + im[5]) + (im[6] + im[7]));
  mpole[(size_t)sp[0] * P + l] = make_double2(r, i);
}

// -------------------------------------------------------------------------
// Downward pass without the level-by-level chain: the local expansion of a
// leaf b is its own (M2L + P2L) part plus the own parts of its ancestors A
// at levels >= 2 shifted directly to its centre (an exact polynomial shift,
// so equal up to rounding to the level-by-level pass).  Scaled form,
// w = (c_b - c_A)/h_A, r = h_b/h_A:
//   c_l += (r/w)^l sum_{k>=l} C(k,l) w^k b_k(A).
// One lane per (leaf, ancestor) pair; a group of <= 8 leaves and <= 64
// pairs per wave; per-leaf sums in pair order through LDS (deterministic).
template <int PM, bool EXACT>
__global__ void __launch_bounds__(64) k_down(int Prt, double root_size, const int* __restrict__ grp,
                                             const int* __restrict__ anc_ptr, const int* __restrict__ anc,
                                             const int* __restrict__ anc_leaf, const int* __restrict__ leaf_box,
                                             const int* __restrict__ box_level, const double* __restrict__ box_cx,
                                             const double* __restrict__ box_cy, const double* __restrict__ pasT,
                                             const double2* __restrict__ local, double2* __restrict__ locf, long smp,
                                             long slf) {
  const int P = EXACT ? PM : Prt;
  local += blockIdx.y * smp;  // right-hand side blockIdx.y
  locf += blockIdx.y * slf;
  __shared__ double2 s_o[8 * kSoStride];
  const int f0 = grp[blockIdx.x], f1 = grp[blockIdx.x + 1];
  const int e0 = anc_ptr[f0], e1 = anc_ptr[f1];
  const int lane = threadIdx.x;
  const int e = e0 + lane;
  const bool act = e < e1;
  const int A = act ? anc[e] : 0;
  const int b = leaf_box[act ? anc_leaf[e] : f0];
  const int la = box_level[A], lb = box_level[b];
  const double hA = box_side(root_size, la);
  const double2 w = act ? make_double2((box_cx[b] - box_cx[A]) / hA, (box_cy[b] - box_cy[A]) / hA)
                        : make_double2(0.5, 0.5);
  const double r = act ? ldexp(1.0, la - lb) : 1.0;
  const double ww = w.x * w.x + w.y * w.y;
  const double2 q = make_double2(r * w.x / ww, -r * w.y / ww);  // r / w
  const int NC = (P + 7) / 8;
  // work-group z computes the outputs l = 8c .. 8c+7 (chunk c = blockIdx.z);
  // the scaled ancestor coefficients s_k = w^k b_k, k >= 8c, are formed on
  // the fly (k outer) rather than held, which keeps the kernel at a few
  // dozen registers
  static_for<0, (PM + 7) / 8>([&](auto cc) __attribute__((always_inline)) {
    constexpr int c = decltype(cc)::value;
    if (c != (int)blockIdx.z || c >= NC) return;
    // q^l before output l: the same product sequence as a running power
    double2 ql = make_double2(1.0, 0.0);
#pragma unroll
    for (int i = 0; i < 8 * c; ++i) ql = cmul(ql, q);
    // w^k from k = 0, the same product sequence as a running power
    double2 pw = make_double2(1.0, 0.0);
#pragma unroll
    for (int k = 0; k < 8 * c; ++k) pw = cmul(pw, w);
    // the eight outputs of the chunk accumulate side by side (k outer)
    double ur[8], ui[8];
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) ur[lc] = ui[lc] = 0.0;
#pragma unroll
    for (int k = 8 * c; k < PM; ++k) {
      const double2 a = (act && k < P) ? local[(size_t)A * P + k] : make_double2(0.0, 0.0);
      const double2 sk = cmul(pw, a);
      pw = cmul(pw, w);
#pragma unroll
      for (int lc = 0; lc < 8; ++lc) {
        const int l = 8 * c + lc;
        if (k >= l && k < P) {
          const double cf = pasT[l * P + k];
          ur[lc] += cf * sk.x;
          ui[lc] += cf * sk.y;
        }
      }
    }
#pragma unroll
    for (int lc = 0; lc < 8; ++lc) {
      const int l = 8 * c + lc;
      double2 out = make_double2(0.0, 0.0);
      if (l < P) {
        out = cmul(ql, make_double2(ur[lc], ui[lc]));
        ql = cmul(ql, q);
      }
      s_o[lc * kSoStride + lane] = act ? out : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int lc = lane & 7, seg = lane >> 3;
    const int f = f0 + seg, l = 8 * c + lc;
    if (f < f1 && l < P) {
      const int bf = leaf_box[f];
      double2 v = make_double2(0.0, 0.0);
      if (box_level[bf] >= 2) {
        const double2 sv = seg_sum(s_o + lc * kSoStride, anc_ptr[f] - e0, anc_ptr[f + 1] - e0);
        const double2 own = local[(size_t)bf * P + l];
        v = make_double2(own.x + sv.x, own.y + sv.y);
      }
      locf[(size_t)f * P + l] = v;
    }
  });
}

// -------------------------------------------------------------------------
// Far field and the near-field reduction: V at every leaf's nodes from its
// full local expansion (L2P), the near field (the row of the same-level
// sources and the rows of the other FP64 list-1 pairs), the M2P rows of list
// 3, all in list order (deterministic), and the log terms: log(h) a_0 of each
// list-1 source and log(h/2) a_0 of each list-3 box.
// Everything is summed in folded form (parity q = 2 qx + qy of a quadrant
// node, values of its four images = signed sums): a lane holds one of the
// H^2 = (K/2)^2 quadrant nodes, so a row is four coalesced loads, and L2P
// needs the powers of one z per lane with real coefficients: with c = a + ib
// and Re(c z^l) = a Re z^l - b Im z^l, the term l adds to parity 0 (a) and 3
// (b) for even l, 2 (a) and 1 (b) for odd l.  That is a quarter of the
// arithmetic of a Horner scheme per node, which took 78% of the vector
// units' time (wedge workload: 39 us alone, now 28).  A wave serves 64 / H^2 leaves (K = 4,
// 8) or one (K = 12, 16), whose coefficients are then wave-uniform.
// NODE: rows in node order too, those of the mixed-precision pairs (y_slot
// holds ~row) and the target-stationary sums (h^2 times the list-1 sum, left
// in V; ts).
// Each row is read once, by its target's wave: those loads are non-temporal.
// (The kernels that write the rows use plain stores, so that part of them is
// still in the last-level cache when this kernel runs; non-temporal stores
// there measured slower.)
struct FarArgs {
  int L, P;
  double root_size;
  bool ts;
  const int *leaf_box, *box_level;
  const double* t;
  const int *l3_ptr, *l3_src, *l3_slot;
  const double* Y3;
  const double2 *locf, *mpole;
  const int *l1_ptr, *l1_srcbox, *sy_row;
  const double* YS;
  const int *y_ptr, *y_slot;
  const double* Y;
  double* V;
  long slf, smp, sys, sny, sy3, sv;
};

template <int K, bool NODE>
__global__ void __launch_bounds__(256) k_far(FarArgs A) {
  constexpr int n = K * K, H = K / 2, H2 = H * H, LPW = H2 <= 16 ? 64 / H2 : 1;
  const long r = blockIdx.y;  // right-hand side
  const double2* __restrict__ locf = A.locf + r * A.slf;
  const double2* __restrict__ mpole = A.mpole + r * A.smp;
  const double* __restrict__ YS = A.YS + r * A.sys;
  const double* __restrict__ Y = A.Y + r * A.sny;
  const double* __restrict__ Y3 = A.Y3 + r * A.sy3;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = LPW > 1 ? lane / H2 : 0;
  const int node = LPW > 1 ? lane % H2 : min(lane, H2 - 1);  // quadrant node
  int leaf = LPW * (4 * blockIdx.x + w) + sub;
  const bool act = leaf < A.L && (LPW > 1 || lane < H2);
  if (LPW * (4 * (int)blockIdx.x + w) >= A.L) return;
  leaf = min(leaf, A.L - 1);
  const int b = A.leaf_box[leaf], lev = A.box_level[b];
  const double h = box_side(A.root_size, lev);
  const int e0 = A.l1_ptr[leaf], n1 = A.l1_ptr[leaf + 1] - e0;
  const int f0 = A.l3_ptr[leaf], n3 = A.l3_ptr[leaf + 1] - f0;
  const int g0 = NODE && A.ts ? 0 : A.y_ptr[leaf], ny = NODE && A.ts ? 0 : A.y_ptr[leaf + 1] - g0;
  const int srow = NODE && A.ts ? -1 : A.sy_row[leaf];
  // log terms: the lanes of a leaf take its sources in turn
  double lg = 0.0, lg3 = 0.0;
  {
    constexpr int G = LPW > 1 ? H2 : 64;
    const int l0 = LPW > 1 ? node : lane;
    for (int e = l0; e < n1; e += G) lg += mpole[(size_t)A.l1_srcbox[e0 + e] * A.P].x;
    for (int e = l0; e < n3; e += G) lg3 += mpole[(size_t)A.l3_src[f0 + e] * A.P].x;
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
      lg += __shfl_xor(lg, o, G);
      lg3 += __shfl_xor(lg3, o, G);
    }
  }
  const double lh = log(h);
  const int na = node / H, nb = node % H;
  const int img[4] = {na * K + nb, na * K + K - 1 - nb, (K - 1 - na) * K + nb, (K - 1 - na) * K + K - 1 - nb};
  double yn[4] = {0.0, 0.0, 0.0, 0.0}, y3[4] = {0.0, 0.0, 0.0, 0.0}, yv[4] = {0.0, 0.0, 0.0, 0.0};
  if (srow >= 0) {
    const double* y = YS + (size_t)srow * n + node;
#pragma unroll
    for (int q = 0; q < 4; ++q) yn[q] = __builtin_nontemporal_load(y + q * H2);
  }
#pragma unroll 4
  for (int e = 0; e < ny; ++e) {
    const int slot = A.y_slot[g0 + e];
    if (NODE && slot < 0) {
      const double* y = Y + (size_t)~slot * n;
#pragma unroll
      for (int k = 0; k < 4; ++k) yv[k] += __builtin_nontemporal_load(y + img[k]);
    } else {
      const double* y = Y + (size_t)slot * n + node;
#pragma unroll
      for (int q = 0; q < 4; ++q) yn[q] += __builtin_nontemporal_load(y + q * H2);
    }
  }
#pragma unroll 4
  for (int e = 0; e < n3; ++e) {
    const double* y = Y3 + (size_t)A.l3_slot[f0 + e] * n + node;
#pragma unroll
    for (int q = 0; q < 4; ++q) y3[q] += __builtin_nontemporal_load(y + q * H2);
  }
  const double h2 = h * h;
#pragma unroll
  for (int q = 0; q < 4; ++q) y3[q] += h2 * yn[q];
  y3[0] += lh * lg + (lh - kLn2) * lg3;
  if (lev >= 2) {
    const double2* __restrict__ c = locf + (size_t)leaf * A.P;
    const double zx = 0.5 * A.t[na], zy = 0.5 * A.t[nb];
    double px = 1.0, py = 0.0;  // z^l
    auto step = [&](int l, double& re, double& im) __attribute__((always_inline)) {
      const double2 cl = c[l];
      re += cl.x * px;
      im -= cl.y * py;
      const double t = px * zx - py * zy;
      py = px * zy + py * zx;
      px = t;
    };
    int l = 0;
#pragma unroll 4
    for (; l + 1 < A.P; l += 2) {
      step(l, y3[0], y3[3]);
      step(l + 1, y3[2], y3[1]);
    }
    if (l < A.P) step(l, y3[0], y3[3]);
  }
  if (act) {
    double* V = A.V + r * A.sv + (size_t)leaf * n;
    if (NODE && A.ts) {
#pragma unroll
      for (int k = 0; k < 4; ++k) yv[k] = V[img[k]];
    } else if (NODE) {
#pragma unroll
      for (int k = 0; k < 4; ++k) yv[k] *= h2;
    }
    const double ep = y3[0] + y3[1], em = y3[0] - y3[1], op = y3[2] + y3[3], om = y3[2] - y3[3];
    const double v[4] = {ep + op, em + om, ep - op, em - om};
#pragma unroll
    for (int k = 0; k < 4; ++k) V[img[k]] = kInv2Pi * (NODE ? v[k] + yv[k] : v[k]);
  }
}

// -------------------------------------------------------------------------
// Values of leaf-grid data at arbitrary points (e.g. boundary nodes): the leaf
// holding a point is found by descending the tree from the root (children in
// Morton order, a point on a box edge goes to the upper/right child); the value
// is the tensor interpolant of the leaf's K x K first-kind Chebyshev samples,
// evaluated by the barycentric formula with weights (-1)^a sin((2a+1)pi/2K).
// Points outside the root box get NaN.
// A wave takes ppw <= 64 points.  Each lane descends the tree for one of them
// (one load per level: box_next is the first child, or ~leaf), then G lanes
// (the power of two >= K) share a point, lane c holding column c of its leaf:
// a row of the leaf is one contiguous load of the group, all K rows are in
// flight together, and each lane forms one weight per axis.  (One thread per
// point read 64 cache lines per load and formed 2K sines: 167 us for 200000
// points at K = 16; now 37 us alone.  The leaves' rows are 391 MB of reads from
// the L2s, 91% hits, about 10 TB/s; the vector units are 43% busy; of the
// waves' time a third is waiting for memory and half for issue.)  The points of a wave are served in turn, so
// ppw is halved until there are kInterpWaves waves, about one full residency
// (200000 points with the net charge after them: 50.4 us for 2048, 45.7 for
// 4096, 44.0 for 8192, 46.9 for 16384).
constexpr int kInterpWaves = 8192;
// v of lane a of the caller's group of G lanes
template <int G, int A>
__device__ __forceinline__ double group_lane(double v) {
  if constexpr (G == 16) {  // a row of the wave: one DPP broadcast per half
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)u, 0x150 + A, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), 0x150 + A, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  } else {
    return __shfl(v, A, G);
  }
}

template <int K>
__global__ void __launch_bounds__(256) k_interp(double root_cx, double root_cy, double root_size,
                                                const int* __restrict__ box_next, const double* __restrict__ t,
                                                const double* __restrict__ V, long npts, int ppw,
                                                const double* __restrict__ px, const double* __restrict__ py,
                                                double* __restrict__ out) {
  constexpr int G = K == 12 ? 16 : K, NG = 64 / G;  // lanes per point, points at a time
  const int lane = threadIdx.x & 63, c = lane & (G - 1), grp = lane / G;
  const long i0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * ppw;
  if (i0 >= npts) return;
  const long i = i0 + lane;
  const bool mine = lane < ppw && i < npts;
  const double x = mine ? px[i] : root_cx, y = mine ? py[i] : root_cy;
  double cx = root_cx, cy = root_cy, h = root_size;
  const bool in = fabs(x - cx) <= 0.5 * h && fabs(y - cy) <= 0.5 * h;  // false for NaN
  int leaf = 0;
  double xi = 0.0, eta = 0.0;
  if (in) {
    int b = box_next[0];
    while (b >= 0) {
      const int dx = x >= cx, dy = y >= cy;
      h *= 0.5;
      cx += (dx ? 0.5 : -0.5) * h;
      cy += (dy ? 0.5 : -0.5) * h;
      b = box_next[b + dx + 2 * dy];
    }
    leaf = ~b;
    xi = 2.0 * (x - cx) / h;
    eta = 2.0 * (y - cy) / h;
  }
  const bool act = c < K;
  const double tc = t[act ? c : 0];
  const double wc = act ? ((c & 1) ? -1.0 : 1.0) * sinpi((2 * c + 1) / (2.0 * K)) : 0.0;
  // this lane's weight of the group's point in one coordinate
  auto weight = [&](double s) {
    const double d = s - tc;
    const bool at = act && d == 0.0;
    const unsigned long long hit = __ballot(at) >> (grp * G) & ((1ull << (G - 1) << 1) - 1);
    double l = wc / (d == 0.0 ? 1.0 : d), sum = l;
#pragma unroll
    for (int o = 1; o < G; o <<= 1) sum += __shfl_xor(sum, o, G);
    return hit ? (at ? 1.0 : 0.0) : l * (1.0 / sum);
  };
  double res = 0.0;
  for (int j0 = 0; j0 < ppw; j0 += NG) {
    const int j = j0 + grp;
    const double* v = V + (size_t)__shfl(leaf, j, 64) * (K * K) + (act ? c : 0);
    double r[K];
#pragma unroll
    for (int a = 0; a < K; ++a) r[a] = v[a * K];
    const double lx = weight(__shfl(xi, j, 64)), ly = weight(__shfl(eta, j, 64));
    double acc = 0.0;
    static_for<0, K>([&](auto ac) __attribute__((always_inline)) {
      acc += group_lane<G, decltype(ac)::value>(lx) * r[decltype(ac)::value];
    });
    acc *= ly;
#pragma unroll
    for (int o = 1; o < G; o <<= 1) acc += __shfl_xor(acc, o, G);
    const double got = __shfl(acc, G * (lane % NG), 64);
    if (lane / NG == j0 / NG) res = got;
  }
  if (mine) out[i] = in ? res : __builtin_nan("");
}

int launch_interp(Plan* p, const double* V, long npts, const double* px, const double* py, double* out,
                  hipStream_t s, std::string& err) {
  Context* c = p->ctx;
  const Tables& T = c->T;
  if (!c->D.ready) {
    int rc = upload_tables(c, err);
    if (rc) return rc;
  }
  if (!p->D.ready) {
    int rc = upload_plan(p, err);
    if (rc) return rc;
  }
  if (npts <= 0) return VFX_OK;
  int ppw = 64;
  const int least = 64 / (T.K == 12 ? 16 : T.K);
  while (ppw > least && (npts + ppw - 1) / ppw < kInterpWaves) ppw /= 2;
  const long blocks = ((npts + ppw - 1) / ppw + 3) / 4;
#define VFX_INTERP(KV)                                                                                             \
  hipLaunchKernelGGL(k_interp<KV>, dim3((unsigned)blocks), dim3(256), 0, s, T.root_cx, T.root_cy, T.root_size,     \
                     p->D.box_next, c->D.t, V, npts, ppw, px, py, out)
  switch (T.K) {
    case 4: VFX_INTERP(4); break;
    case 8: VFX_INTERP(8); break;
    case 12: VFX_INTERP(12); break;
    default: VFX_INTERP(16); break;
  }
#undef VFX_INTERP
  VFX_HIP(hipGetLastError());
  return VFX_OK;
}

// -------------------------------------------------------------------------
// Net charge A^e = integral of f^e over the tree (Section 6, exterior
// problem: the volume potential then grows like A^e log|x|, which the
// boundary solve must offset).  Each leaf contributes h^2 sum_j w_j f_j with
// w the tensor first-kind Chebyshev (Fejer) weights of the unit square.  Two
// passes with a fixed partition, so the sum order depends on the tree only:
// block b of right-hand side r sums the nodes of leaves [b L/G, (b+1) L/G)
// (each thread a strided share, then a fixed LDS tree) into part[r G + b];
// one block per right-hand side then sums its G partials the same way
// (thread t the partials t, t + 256, ... in order).  G is about L n / 2048
// (eight samples per thread, enough loads in flight without flooding the
// dispatcher with tiny blocks), at least 1 and at most min(L, 2048).
constexpr int kChargeBlocks = 2048;

__device__ __forceinline__ double block_sum_256(double v, double* red) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
#pragma unroll
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  return red[0];
}

__global__ void __launch_bounds__(256) k_charge_part(int n, int L, int G, double root_size,
                                                     const int* __restrict__ leaf_box, const int* __restrict__ box_level,
                                                     const double* __restrict__ w2, const double* __restrict__ fe,
                                                     long sfe, double* __restrict__ part) {
  __shared__ double red[256];
  fe += blockIdx.y * sfe;
  const int b = blockIdx.x;
  const long l0 = (long)b * L / G, l1 = (long)(b + 1) * L / G;
  double acc = 0.0;
  for (long i = l0 * n + threadIdx.x; i < l1 * n; i += 256) {
    const int leaf = (int)(i / n), j = (int)(i - (long)leaf * n);
    const double h = box_side(root_size, box_level[leaf_box[leaf]]);
    acc += h * h * w2[j] * fe[i];
  }
  const double s = block_sum_256(acc, red);
  if (threadIdx.x == 0) part[(size_t)blockIdx.y * G + b] = s;
}

__global__ void __launch_bounds__(256) k_charge_sum(int G, const double* __restrict__ part, double* __restrict__ out) {
  __shared__ double red[256];
  double v = 0.0;
  for (int q = threadIdx.x; q < G; q += 256) v += part[(size_t)blockIdx.x * G + q];
  const double s = block_sum_256(v, red);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

int launch_net_charge(Plan* p, const double* fe, int nrhs, double* out, hipStream_t s, std::string& err) {
  Context* c = p->ctx;
  const Tables& T = c->T;
  if (!c->D.ready) {
    int rc = upload_tables(c, err);
    if (rc) return rc;
  }
  if (!p->D.ready) {
    int rc = upload_plan(p, err);
    if (rc) return rc;
  }
  DevicePlan& D = p->D;
  const int L = p->H.L, n = T.n;
  const int G = std::min(L, (int)std::max(1L, std::min((long)kChargeBlocks, (long)L * n / 2048)));
  if (nrhs > D.chg_cap) {
    p->gen++;  // graphs that captured the old buffer are stale
    if (D.chg_part) {
      VFX_HIP(hipDeviceSynchronize());  // no earlier call of this plan in flight
      VFX_HIP(hipFree(D.chg_part));
      D.chg_part = nullptr;
      D.chg_cap = 0;
    }
    VFX_HIP(hipMalloc((void**)&D.chg_part, sizeof(double) * kChargeBlocks * (size_t)nrhs));
    D.chg_cap = nrhs;
  }
  if (G > 0)
    hipLaunchKernelGGL(k_charge_part, dim3(G, nrhs), dim3(256), 0, s, n, L, G, T.root_size, D.leaf_box,
                       D.box_level, c->D.w2, fe, (long)L * n, D.chg_part);
  VFX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_charge_sum, dim3(nrhs), dim3(256), 0, s, G, D.chg_part, out);
  VFX_HIP(hipGetLastError());
  return VFX_OK;
}

// -------------------------------------------------------------------------
// Net charge without allocation (for callers that cannot allocate: code
// under HIP graph capture, tight serving loops).  The block partials go to
// a file-scope device array instead of the plan's buffer: one copy per GPU
// for the life of the process, kNoallocMaxRhs right-hand sides of
// kChargeBlocks partials (1 MiB).  Host code never names the array in a
// launch or a copy: on each device it asks hipGetSymbolAddress for that
// device's copy once (with the device current) and passes the address it
// returns.  Every partial the sum reads is written by the same call first,
// so nothing needs clearing; two calls that overlap on one GPU race on it.
constexpr int kNoallocMaxRhs = 64;
static __device__ __align__(256) double scratch[kChargeBlocks * kNoallocMaxRhs];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static int scratch_address(int dev, void** out, std::string& err) {
  if (dev < 0 || dev >= kMaxDevices) {
    err = "device ordinal out of range";
    return VFX_EINVAL;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    VFX_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) {
      err = "hipGetSymbolAddress returned a null address";
      return VFX_EHIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return VFX_OK;
}

int noalloc_max_rhs() { return kNoallocMaxRhs; }

int launch_net_charge_noalloc(Plan* p, const double* fe, int nrhs, double* out, hipStream_t s, std::string& err) {
  Context* c = p->ctx;
  if (!c->D.ready || !p->D.ready) {
    err = "the plan's device data are not resident (run vfx_execute or vfx_net_charge on it once first)";
    return VFX_EINVAL;
  }
  if (nrhs > kNoallocMaxRhs) {
    err = "nrhs exceeds the allocation-free limit of " + std::to_string(kNoallocMaxRhs);
    return VFX_EINVAL;
  }
  int dev = -1;
  VFX_HIP(hipGetDevice(&dev));
  if (dev != c->D.device) {
    err = "the current device is not the one holding the plan's data";
    return VFX_EINVAL;
  }
  void* ptr = nullptr;
  int rc = scratch_address(dev, &ptr, err);
  if (rc) return rc;
  double* part = static_cast<double*>(ptr);
  const Tables& T = c->T;
  const DevicePlan& D = p->D;
  const int L = p->H.L, n = T.n;
  const int G = std::min(L, (int)std::max(1L, std::min((long)kChargeBlocks, (long)L * n / 2048)));
  if (G > 0)
    hipLaunchKernelGGL(k_charge_part, dim3(G, nrhs), dim3(256), 0, s, n, L, G, T.root_size, D.leaf_box,
                       D.box_level, c->D.w2, fe, (long)L * n, part);
  VFX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_charge_sum, dim3(nrhs), dim3(256), 0, s, G, part, out);
  VFX_HIP(hipGetLastError());
  return VFX_OK;
}

// -------------------------------------------------------------------------
template <typename T>
static int upload(T** dst, const T* src, size_t count, std::string& err) {
  *dst = nullptr;
  if (count == 0) return VFX_OK;
  VFX_HIP(hipMalloc((void**)dst, count * sizeof(T)));
  VFX_HIP(hipMemcpy(*dst, src, count * sizeof(T), hipMemcpyHostToDevice));
  return VFX_OK;
}

#define UP(dst, vec)                                                       \
  do {                                                                     \
    int rc_ = upload(&(dst), (vec).data(), (vec).size(), err);             \
    if (rc_) return rc_;                                                   \
  } while (0)

// Rows of K^2 target nodes in folded form: y_q of a quadrant node is a quarter
// of the signed sum of its four images (q = 2 qx + qy).
static std::vector<double> fold_rows(const std::vector<double>& v, int K) {
  const int n = K * K, H = K / 2, H2 = H * H;
  std::vector<double> o(v.size());
  for (size_t r = 0; r + n <= v.size(); r += n)
    for (int i = 0; i < H2; ++i) {
      const int a = i / H, b = i % H, a1 = K - 1 - a, b1 = K - 1 - b;
      const long double y0 = v[r + a * K + b], y1 = v[r + a * K + b1], y2 = v[r + a1 * K + b], y3 = v[r + a1 * K + b1];
      o[r + i] = (double)((y0 + y1 + y2 + y3) / 4);
      o[r + H2 + i] = (double)((y0 - y1 + y2 - y3) / 4);
      o[r + 2 * H2 + i] = (double)((y0 + y1 - y2 - y3) / 4);
      o[r + 3 * H2 + i] = (double)((y0 - y1 - y2 + y3) / 4);
    }
  return o;
}

int upload_tables(Context* c, std::string& err) {
  const Tables& T = c->T;
  DeviceTables& D = c->D;
  UP(D.t, T.t);
  UP(D.w2, T.w2);
  UP(D.AbarT, T.AbarT);
  UP(D.A, T.A);
  UP(D.cbar, T.cbar);
  UP(D.mom_T, T.mom_T);
  UP(D.sym_T, T.sym_T);
  const std::vector<double> pair_f = fold_rows(T.pair_T, T.K), m2p_f = fold_rows(T.m2p_gemm, T.K);
  UP(D.pair_T, pair_f);
  UP(D.lr_R, T.lr_R);
  UP(D.fx_W, T.fx_W);
  UP(D.fx_Wexp, T.fx_Wexp);
  if (T.ts_ok) {
    UP(D.cls_R, T.cls_R);
    UP(D.lr_Wp, T.lr_Wp);
    UP(D.cls_QT, T.cls_QT);
    UP(D.self_T, T.self_T);
  }
  UP(D.fx_Q, T.fx_Q);
  UP(D.fx_Qexp, T.fx_Qexp);
  UP(D.fx_A, T.fx_A);
  UP(D.fx_Aexp, T.fx_Aexp);
  UP(D.f8_W, T.f8_W);
  UP(D.f8_Wexp, T.f8_Wexp);
  UP(D.f8_Q, T.f8_Q);
  UP(D.f8_Qexp, T.f8_Qexp);
  UP(D.f8_A, T.f8_A);
  UP(D.f8_Aexp, T.f8_Aexp);
  UP(D.p2l_gemm, T.p2l_gemm);
  UP(D.m2p_gemm, m2p_f);
  UP(D.pas_m2l_t, T.pas_m2l_t);
  UP(D.pas_m2m_t, T.pas_m2m_t);
  UP(D.pas_l2l_t, T.pas_l2l_t);
  UP(D.m2l_logd, T.m2l_logd);
  VFX_HIP(hipGetDevice(&D.device));
  D.ready = true;
  return VFX_OK;
}

void free_tables_device(Context* c) {
  DeviceTables& D = c->D;
  c->gen++;
  void* ptrs[] = {D.t, D.w2, D.AbarT, D.cbar, D.mom_T, D.sym_T, D.pair_T, D.A, D.m2l_logd, D.p2l_gemm, D.m2p_gemm,
                  D.pas_m2l_t, D.pas_m2m_t, D.pas_l2l_t, D.lr_R, D.fx_W, D.fx_Q, D.fx_A, D.fx_Wexp, D.fx_Qexp,
                  D.fx_Aexp, D.f8_W, D.f8_Q, D.f8_A, D.f8_Wexp, D.f8_Qexp, D.f8_Aexp, D.cls_R, D.lr_Wp, D.cls_QT,
                  D.self_T};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  D = DeviceTables();
}

// Buffers that hold one copy per right-hand side (expansions, moments,
// near-field, P2L and M2P rows, leaf local expansions, slices, the batched
// extension's products): this one list is what a larger batch reallocates and
// what goes with the plan's device data.
static void free_rhs_buffers(DevicePlan& D) {
  void* bufs[] = {D.mpole, D.local, D.mom,  D.ysym,   D.near_y, D.near_z, D.p2l_y, D.m2p_y,
                  D.up_part, D.locf, D.xs, D.xs_exp, D.ext_fg, D.ext_g};
  for (void* q : bufs)
    if (q) (void)hipFree(q);
  D.mpole = D.local = D.up_part = D.locf = nullptr;
  D.mom = D.ysym = D.near_y = D.near_z = D.p2l_y = D.m2p_y = nullptr;
  D.xs = nullptr;
  D.xs_exp = nullptr;
  D.ext_fg = D.ext_g = nullptr;
  D.cap = 0;
}

int ensure_rhs_capacity(Plan* p, int nrhs, std::string& err) {
  const HostPlan& H = p->H;
  DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  const size_t P = T.p + 1, R = (size_t)nrhs;
  if (D.cap > 0) (void)hipDeviceSynchronize();  // no execute of this plan in flight
  p->gen++;  // graphs that captured the old buffers are stale
  free_rhs_buffers(D);
  VFX_HIP(hipMalloc((void**)&D.mpole, sizeof(double2) * (size_t)H.B * P * R));
  VFX_HIP(hipMalloc((void**)&D.local, sizeof(double2) * (size_t)H.B * P * R));
  VFX_HIP(hipMemset(D.local, 0, sizeof(double2) * (size_t)H.B * P * R));
  {
    // moments; the row past the leaves is the zero source
    const size_t wm = sizeof(double) * 4 * moment_stride(T.mom_E), rows = (size_t)H.L + 1;
    VFX_HIP(hipMalloc((void**)&D.mom, wm * rows * R));
    VFX_HIP(hipMemset2D((char*)D.mom + wm * H.L, wm * rows, 0, wm, R));
  }
  if (!H.sy_tgt.empty()) VFX_HIP(hipMalloc((void**)&D.ysym, sizeof(double) * H.sy_tgt.size() * T.n * R));
  if (!H.np_src.empty() && !H.ts) VFX_HIP(hipMalloc((void**)&D.near_y, sizeof(double) * H.np_src.size() * T.n * R));
  if (!H.np_src.empty() && H.ts)
    VFX_HIP(hipMalloc((void**)&D.near_z, sizeof(double) * H.np_src.size() * kNearLrMax * R));
  if (!H.p4_src.empty()) VFX_HIP(hipMalloc((void**)&D.p2l_y, sizeof(double) * H.p4_src.size() * T.p2l_rows * R));
  if (!H.p3_src.empty()) VFX_HIP(hipMalloc((void**)&D.m2p_y, sizeof(double) * H.p3_src.size() * T.n * R));
  if (H.up_slots > 0) VFX_HIP(hipMalloc((void**)&D.up_part, sizeof(double2) * (size_t)H.up_slots * P * R));
  VFX_HIP(hipMalloc((void**)&D.locf, sizeof(double2) * (size_t)H.L * P * R));
  if (H.precision >= 1 && !H.ts) {  // bf16 slices (mode 1) or int8 slices (mode 2, 5/8 of the size)
    VFX_HIP(hipMalloc((void**)&D.xs, sizeof(uint16_t) * 4 * (size_t)H.L * T.n * R));
    VFX_HIP(hipMalloc((void**)&D.xs_exp, sizeof(int) * (size_t)H.L * R));
  }
  if (nrhs >= kExtGemmMinRhs && H.ncut > 0) {
    VFX_HIP(hipMalloc((void**)&D.ext_fg, sizeof(double) * (size_t)H.ncut * R * T.nG));
    VFX_HIP(hipMalloc((void**)&D.ext_g, sizeof(double) * (size_t)H.ncut * R * T.Kbar * T.Kbar));
  }
  // the fills above run on the null stream, which the executes' streams need
  // not wait for
  VFX_HIP(hipStreamSynchronize(nullptr));
  D.cap = nrhs;
  return VFX_OK;
}

int upload_plan(Plan* p, std::string& err) {
  const HostPlan& H = p->H;
  DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  const int P = T.p + 1;
  UP(D.box_level, H.box_level);
  {
    // first child of a box, ~leaf of a leaf box
    std::vector<int> next(H.B);
    for (int b = 0; b < H.B; ++b) next[b] = H.box_leaf[b] >= 0 ? ~H.box_leaf[b] : H.box_child0[b];
    UP(D.box_next, next);
  }
  UP(D.box_cx, H.box_cx);
  UP(D.box_cy, H.box_cy);
  UP(D.leaf_box, H.leaf_box);
  {
    // where each leaf's f^e comes from: 2 an extension list, 1 f (regular), 0 zero
    std::vector<int8_t> src(H.L, 0);
    for (int i = 0; i < H.L; ++i) src[i] = H.owner[i] >= 0 ? 2 : (H.kind[i] == 1 ? 1 : 0);
    UP(D.fe_src, src);
  }
  UP(D.l1_ptr, H.l1_ptr);
  UP(D.l1_srcbox, H.l1_srcbox);
  UP(D.l2_ptr, H.l2_ptr);
  UP(D.l2_src, H.l2_src);
  UP(D.l2_off, H.l2_off);
  UP(D.l2_tgt, H.l2_tgt);
  UP(D.m2l_grp, H.m2l_grp);
  UP(D.l3_ptr, H.l3_ptr);
  UP(D.l3_src, H.l3_src);
  UP(D.anc_ptr, H.anc_ptr);
  UP(D.anc, H.anc);
  UP(D.anc_leaf, H.anc_leaf);
  UP(D.dn_grp, H.dn_grp);

  UP(D.up_box, H.up_box);
  UP(D.up_ptr, H.up_ptr);
  UP(D.up_src, H.up_src);
  UP(D.up_pos, H.up_pos);
  UP(D.up_grp, H.up_grp);
  UP(D.up_split, H.up_split);
  UP(D.l4_ptr, H.l4_ptr);
  UP(D.l4_src, H.l4_src);
  UP(D.np_src, H.np_src);
  UP(D.y_ptr, H.y_ptr);
  UP(D.y_slot, H.y_slot);
  UP(D.sy_nb, H.sy_nb);
  UP(D.sy_row, H.sy_row);
  UP(D.nl_cfg, H.nl_cfg);
  UP(D.nl_first, H.nl_first);
  UP(D.nl_count, H.nl_count);
  UP(D.mt_cfg, H.mt_cfg);
  UP(D.mt_first, H.mt_first);
  UP(D.mt_count, H.mt_count);
  UP(D.ml_cfg, H.ml_cfg);
  UP(D.ml_first, H.ml_first);
  UP(D.ml_count, H.ml_count);
  UP(D.ts_grp, H.ts_grp);
  UP(D.ts_tcls, H.ts_tcls);
  UP(D.ts_row, H.ts_row);
  UP(D.ts_code, H.ts_code);

  UP(D.p4_src, H.p4_src);
  UP(D.l4_slot, H.l4_slot);
  UP(D.t4_cfg, H.t4_cfg);
  UP(D.t4_first, H.t4_first);
  UP(D.t4_count, H.t4_count);
  UP(D.p3_src, H.p3_src);
  UP(D.l3_slot, H.l3_slot);
  UP(D.t3_cfg, H.t3_cfg);
  UP(D.t3_first, H.t3_first);
  UP(D.t3_count, H.t3_count);
  UP(D.leaf_ids, H.leaf_ids);

  UP(D.ext_ptr, H.ext_ptr);
  UP(D.ext_tgt, H.ext_tgt);
  UP(D.ext_geo, H.ext_geo);
  UP(D.pinv_ptr, H.pinv_ptr);
  UP(D.pinv_idx, H.pinv_idx);
  if (H.factored) {
    UP(D.pinv_val, H.pinv_val);
  } else if (H.ncut > 0) {
    VFX_HIP(hipMalloc((void**)&D.pinv_val, sizeof(double) * (size_t)H.pinv_ptr[H.ncut] * T.nG));
  }
  D.factored = H.factored;
  UP(D.sbar_given, H.sbar_given);
  D.cap = 0;
  {
    int rc = ensure_rhs_capacity(p, 1, err);
    if (rc) return rc;
  }
  VFX_HIP(hipStreamCreateWithFlags(&p->side, hipStreamNonBlocking));
  VFX_HIP(hipEventCreateWithFlags(&p->fork_ev, hipEventDisableTiming));
  VFX_HIP(hipEventCreateWithFlags(&p->join_ev, hipEventDisableTiming));
  VFX_HIP(hipEventCreateWithFlags(&p->p2l_ev, hipEventDisableTiming));
  VFX_HIP(hipEventCreateWithFlags(&p->up_ev, hipEventDisableTiming));
  VFX_HIP(hipEventCreateWithFlags(&p->mom_ev, hipEventDisableTiming));
  D.ready = true;
  return VFX_OK;
}

void free_plan_device(Plan* p) {
  DevicePlan& D = p->D;
  if (D.ready) (void)hipDeviceSynchronize();  // no execute of this plan in flight
  p->gen++;
  free_rhs_buffers(D);
  void* ptrs[] = {D.box_level, D.box_next, D.box_cx, D.box_cy, D.leaf_box, D.l1_ptr, D.l2_ptr, D.l2_src, D.l2_off,
                  D.l3_ptr, D.l3_src, D.l4_ptr, D.l4_src, D.np_src, D.y_ptr, D.y_slot, D.sy_nb, D.sy_row, D.p4_src,
                  D.l4_slot, D.t4_cfg, D.t4_first, D.t4_count, D.ext_ptr, D.ext_tgt, D.pinv_ptr, D.pinv_idx,
                  D.pinv_val, D.sbar_given, D.leaf_ids, D.l2_tgt, D.m2l_grp, D.up_box, D.up_ptr, D.up_src, D.up_pos,
                  D.up_split, D.up_grp, D.anc_ptr, D.anc, D.nl_cfg, D.nl_first, D.nl_count, D.l1_srcbox, D.ext_geo,
                  D.anc_leaf, D.dn_grp, D.mt_cfg, D.mt_first, D.mt_count, D.ml_cfg, D.fac_ws, D.ml_first, D.ml_count,
                  D.p3_src, D.l3_slot, D.t3_cfg, D.t3_first, D.t3_count, D.chg_part, D.ts_grp, D.ts_tcls, D.ts_row,
                  D.ts_code, D.fe_src};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  D = DevicePlan();
  for (auto& e : p->ev)
    if (e) (void)hipEventDestroy(e);
  p->ev.clear();
  p->n_timed = 0;
  if (p->side) (void)hipStreamSynchronize(p->side);
  if (p->fork_ev) (void)hipEventDestroy(p->fork_ev);
  if (p->join_ev) (void)hipEventDestroy(p->join_ev);
  if (p->p2l_ev) (void)hipEventDestroy(p->p2l_ev);
  if (p->up_ev) (void)hipEventDestroy(p->up_ev);
  if (p->mom_ev) (void)hipEventDestroy(p->mom_ev);
  if (p->side) (void)hipStreamDestroy(p->side);
  p->fork_ev = p->join_ev = p->p2l_ev = p->up_ev = p->mom_ev = nullptr;
  p->side = nullptr;
}

// Grid of a persistent, XCD-aware kernel: at most max_wgs work-groups (0 =
// one per item), but never fewer than min(items, 8) - the kernels split
// their items into eight contiguous ranges walked by the work-groups of one
// XCD each (blockIdx % 8), so every range needs a work-group.
static int persistent_grid(int items, int max_wgs) {
  int grid = (max_wgs > 0 && items > max_wgs) ? max_wgs : items;
  return std::max(grid, std::min(items, 8));
}

template <int KD, int MTB>
static void launch_gemm(int ntiles, int MT, const int* cfg, const int* first, const int* count, const int* src,
                        const double* A, const double* X, double* Y, hipStream_t s, int max_wgs, unsigned R, long sx,
                        long sy, int ldx = KD, int kx = KD) {
  const int items = ntiles * (MT / MTB);
  const int grid = persistent_grid(items, max_wgs);
  hipLaunchKernelGGL((k_tgemm<KD, MTB>), dim3(grid, R), dim3(256), 0, s, items, MT, cfg, first, count, src, A, X, Y,
                     sx, sy, ldx, kx);
}

// M2P tables: contraction over the 2P real coefficients of a multipole
// (padded to KD = 64 or 128), n = K^2 rows in blocks as for the dense near
// field.
static void m2p_gemm(int n, int kd, int P2, int ntiles, const int* cfg, const int* first, const int* count,
                     const int* src, const double* A, const double* X, double* Y, hipStream_t s, unsigned R, long sx,
                     long sy) {
  if (ntiles <= 0) return;
  const int MT = n / 16;
#define VFX_M2P(KDV, MTBV)                                                                                        \
  launch_gemm<KDV, MTBV>(ntiles, MT, cfg, first, count, src, A, X, Y, s, 0, R, sx, sy, P2, P2)
#define VFX_M2P_N(KDV)            \
  switch (n) {                    \
    case 16: VFX_M2P(KDV, 1); break;  \
    case 64: VFX_M2P(KDV, 4); break;  \
    case 144: VFX_M2P(KDV, 9); break; \
    default: VFX_M2P(KDV, 4); break;  \
  }
  if (kd == 64) {
    VFX_M2P_N(64)
  } else {
    VFX_M2P_N(128)
  }
#undef VFX_M2P_N
#undef VFX_M2P
}

// Leaves times right-hand sides from which the side stream is used: about where
// it pays at K = 16 and p = 24.  One and two streams, us per execute of one
// right-hand side:
//   K = 16, p = 24   376 leaves 74, 91; 808: 89, 96; 976: 97, 99; 1114: 100, 98;
//                    1840: 118, 110; 4198: 148, 135
//   K = 16, p = 40   376: 101, 103; 532: 105, 106; 808: 124, 112; 976: 128, 117
//   K = 12, p = 30   532: 87, 94; 850: 101, 97; 2056: 129, 116; 4204: 156, 137
//   K = 8, p = 20    1495 to 1741: 71-75, 90-96; 2929: 93, 95; 4546: 100, 100
//   K = 4, p = 17    472: 79, 93; 1696: 85, 98; 5788: 172, 181; 20668: 383, 388
// and batches: 502 leaves x 5 at K = 12 159, 129; 136 x 7 at K = 16 110, 110, x
// 12 212, 207; 145 x 7 at K = 8 85, 101, x 12 152, 160.  The near field grows
// like K^4, the waits do not: at K <= 8 the tie is past 4000 leaves (the waits
// of the two-stream form vary there from run to run by 20 us), at p = 40 near
// 600.
constexpr long kTwoStreamLeaves = 1000;
// The same with mixed pairs.  The bf16 kernel takes 45 us and more on the
// smallest trees, so it is worth hiding behind M2L as soon as that is long:
// from leaves times P^2 of 250000 on (one and two streams: p = 20, 256 leaves
// 90 and 105 us, 808 leaves 125 and 118; p = 24, 256 leaves 92 and 110, 532
// leaves 124 and 115; p = 30, 376 leaves 126 and 119; p = 40, 376 leaves 148
// and 120), and for every tree whose order has no compile-time M2L (p = 27, 64
// leaves 138 and 111 us, 976 leaves 196 and 163).  The int8 kernel is shorter:
// as FP64, but for those orders from 400 leaves on (p = 17, 256 leaves 93 and
// 101 us, 808 leaves 130 and 121; p = 27, 532 leaves 150 and 143).
constexpr long kTwoStreamBf16Work = 250000, kTwoStreamInt8General = 400;
// expansion lengths P with a compile-time M2L (k_m2l_lanes)
static bool m2l_lanes(int P) { return P == 21 || P == 25 || P == 31 || P == 41; }
static bool one_stream(long leaves, int P, int mixed_mode) {
  if (mixed_mode == 1) return m2l_lanes(P) && leaves * P * P < kTwoStreamBf16Work;
  if (mixed_mode == 2 && !m2l_lanes(P)) return leaves < kTwoStreamInt8General;
  return leaves < kTwoStreamLeaves;
}
// Below this many leaves the bf16 slices are cut after the moments and P2L
// runs on the caller's stream; from it on they are cut beside the moments and
// P2L runs ahead of the near field.  us per execute of the two: 4198 leaves
// p = 20 161 and 170, p = 24 165 and 170, p = 30 188 and 195; 2050 leaves p =
// 24 135 and 143; 10558 leaves p = 24 279 and 283; 14254 leaves p = 20 401 and
// 357, p = 24 380 and 375.  (Slices beside the moments with P2L on the
// caller's stream, as for int8: 183, 183, 208; 133; 299; 368, 378.)
constexpr int kBf16SlicesFirst = 12000;
// list-2 groups times right-hand sides up to which the compile-time M2L runs
// one work-group per chunk of outputs: two groups per CU, beyond which the
// chunks' repeated source loads cost more than the idle CUs.  Split and not, us
// per execute: p = 24, 32 to 306 groups 69-97, 73-99; p = 40, 32 groups 92, 106;
// 306: 129, 137; 344: 120, 127; 444: 141, 142; p = 30, 312: 103, 102; ten trees
// of 160 to 976 leaves 778, 824; p = 24, 1313 groups (4207 leaves, with the
// limit at 2000) 163, 139.
constexpr long kM2LSplitGroups = 512;

int launch_execute(Plan* p, int nrhs, const double* f_leaf, const double* f_cut, double* fe, double* V,
                   hipStream_t s, std::string& err) {
  Context* c = p->ctx;
  const Tables& T = c->T;
  if (!c->D.ready) {
    int rc = upload_tables(c, err);
    if (rc) return rc;
  }
  if (!p->D.ready) {
    int rc = upload_plan(p, err);
    if (rc) return rc;
  }
  if (nrhs > p->D.cap) {
    int rc = ensure_rhs_capacity(p, nrhs, err);
    if (rc) return rc;
  }
  if (!p->D.factored) {
    err = "the plan defers its least-squares operators to the GPU: call vfx_plan_factor_gpu first";
    return VFX_EINVAL;
  }
  const HostPlan& H = p->H;
  const DeviceTables& DT = c->D;
  const DevicePlan& D = p->D;
  const int n = T.n, P = T.p + 1, L = H.L;
  // per-right-hand-side strides (elements) of the batched buffers
  const long sFL = (long)L * n, sFC = (long)H.ncut * T.nX, sMP = (long)H.B * P;
  const long sNY = (long)H.np_src.size() * n, sYS = (long)H.sy_tgt.size() * n, sPL = (long)H.p4_src.size() * T.p2l_rows;
  const long sNZ = (long)H.np_src.size() * kNearLrMax;
  const long sM3 = (long)H.p3_src.size() * n;
  const long sUP = (long)H.up_slots * P, sLF = (long)L * P;
  const unsigned R = (unsigned)nrhs;
    constexpr int kMaxTimed = 4096;
  constexpr int NE = Plan::kEvents;
  const bool timed = p->timing && p->n_timed < kMaxTimed;
  const size_t ev0 = (size_t)p->n_timed * NE;
  if (timed && p->ev.size() < ev0 + NE) {
    for (int k = 0; k < NE; ++k) {
      hipEvent_t e;
      VFX_HIP(hipEventCreate(&e));
      p->ev.push_back(e);
    }
  }
  if (timed) p->ev_set.resize(p->n_timed + 1), p->ev_set.back() = 0;
  auto mark = [&](int k, hipStream_t st) -> int {
    if (timed) {
      p->ev_set[p->n_timed] |= 1u << k;
      hipError_t e = hipEventRecord(p->ev[ev0 + k], st);
      if (e != hipSuccess) {
        err = std::string("hipEventRecord: ") + hipGetErrorString(e);
        return VFX_EHIP;
      }
    }
    return VFX_OK;
  };
#define MARK(k, st)          \
  do {                       \
    int rc_ = mark(k, st);   \
    if (rc_) return rc_;     \
  } while (0)
  MARK(Plan::evStart, s);
  {
    // the extension of every cut leaf, and in the same launch the f^e
    // initialisation of the other leaves
    const int ext_blocks = H.ncut * nrhs;
    const long pieces = (long)L * n / 2 * nrhs;
    // a batch of at least kExtGemmMinRhs right-hand sides: A1 and A2 as
    // MFMA GEMMs, then the Chebyshev step and the evaluation for eight
    // right-hand sides per work-group; the extension kernel only
    // initialises the leaves no extension list writes
    const bool gemm = nrhs >= kExtGemmMinRhs && H.ncut > 0;
    if (gemm) {
      int rc = launch_ext_gemm(p, f_cut, nrhs, s, err);
      if (!rc) rc = launch_ext_eval(p, f_cut, fe, nrhs, s, err);
      if (rc) return rc;
    }
    const int blocks1 = gemm ? 0 : ext_blocks;
    const int nt = blocks1 > 0 && blocks1 <= kExtOnePerCu ? 1024 : 256;
    const int copy_blocks = (int)std::min<long>((pieces + nt - 1) / nt, 262144 / nt);
#define VFX_EXT(NTV)                \
  if (T.Kbar != 12)                 \
    VFX_EXTK(NTV, 0, 0);            \
  else if (T.K == 16)               \
    VFX_EXTK(NTV, 16, 12);          \
  else if (T.K == 12)               \
    VFX_EXTK(NTV, 12, 12);          \
  else if (T.K == 8)                \
    VFX_EXTK(NTV, 8, 12);           \
  else                              \
    VFX_EXTK(NTV, 4, 12)
#define VFX_EXTK(NTV, KV, KBV)                                                                                     \
  hipLaunchKernelGGL((k_extension<NTV, KV, KBV>), dim3(blocks1 + copy_blocks), dim3(NTV), 0, s, T.K, T.Kbar, T.nX, T.nG,      \
                     D.pinv_ptr, D.pinv_idx, D.pinv_val, D.sbar_given, D.ext_ptr, D.ext_tgt, D.ext_geo, DT.t,      \
                     DT.AbarT, DT.cbar, f_cut, fe, nrhs, sFC, sFL, blocks1, L, D.fe_src, f_leaf)
    if (nt == 1024) {
      VFX_EXT(1024);
    } else {
      VFX_EXT(256);
    }
#undef VFX_EXT
#undef VFX_EXTK
  }
  VFX_HIP(hipGetLastError());
  MARK(Plan::evExt, s);
  // fork: P2L and the near field on the side stream, concurrent with the
  // upward pass, M2L and the downward pass on the caller's stream.  The
  // persistent near-field grids are bounded (about two work-groups per CU,
  // looping over the tiles).  The side stream starts after the moments, or
  // beside them if the slices of a mixed near field are cut there.
  // Small trees stay on the caller's stream: a wait between streams costs
  // about 7 us, more than their near field takes beside the other kernels.
  const bool mixed = H.precision >= 1 && !H.ts && !(H.ml_cfg.empty() && H.mt_cfg.empty());
  const bool one = !H.ts && one_stream((long)L * nrhs, P, mixed ? H.precision : 0);
  hipStream_t side = one ? s : p->side;
  const bool slices_late = mixed && H.precision == 1 && L < kBf16SlicesFirst;
  const bool p2l_caller = mixed && (H.precision == 2 || slices_late);  // else on the side stream
  auto split = [&]() -> int {
    MARK(Plan::evSlice0, side);
    int rc = H.precision == 2 ? launch_split_f8(p, fe, nrhs, side, err) : launch_split_fx(p, fe, nrhs, side, err);
    if (!rc) rc = mark(Plan::evSlice1, side);
    return rc;
  };
  auto p2l = [&](hipStream_t st) -> int {
    if (H.t4_cfg.empty()) return VFX_OK;
    MARK(Plan::evP2l0, st);
    int rc = launch_p2l(p, nrhs, st, err);
    if (!rc) rc = mark(Plan::evP2l1, st);
    return rc;
  };
  if (mixed && !slices_late) {
    if (!one) {
      VFX_HIP(hipEventRecord(p->fork_ev, s));
      VFX_HIP(hipStreamWaitEvent(side, p->fork_ev, 0));
    }
    int rc = split();
    if (rc) return rc;
  }
  // exterior moments and multipoles of the leaves
  MARK(Plan::evMom0, s);
  {
    int rc = launch_moments(p, fe, nrhs, s, err);
    if (rc) return rc;
  }
  MARK(Plan::evMom1, s);
  if (!one) {
    VFX_HIP(hipEventRecord(p->mom_ev, s));
    VFX_HIP(hipStreamWaitEvent(side, p->mom_ev, 0));
  }
  if (slices_late) {
    int rc = split();
    if (rc) return rc;
  }
  // P2L first on the side stream (M2L on the caller's stream waits for it),
  // then the near field.  With a mixed near field P2L mostly runs before M2L
  // on the caller's stream instead: the mixed kernel holds its full register
  // file and is best started beside the upward pass (14254 leaves, int8: 337
  // -> 323 us; bf16: kBf16SlicesFirst); the FP64 near field is better after
  // P2L (the same tree: 259 against 263 us).
  if (H.nlev > 2 && !p2l_caller) {
    int rc = p2l(side);
    if (rc) return rc;
  }
  if (!one && !p2l_caller) VFX_HIP(hipEventRecord(p->p2l_ev, side));
  if (H.ts) {
    // target-stationary near field: the factor products Z = (W_b P_g^T) f
    // of every non-self pair (table GEMM over the configuration-major
    // tiles), then the per-target-group kernel, which leaves h^2 times each
    // leaf's list-1 table sum in V
    MARK(Plan::evNear0, side);
    if (!H.nl_cfg.empty())
      launch_gemm<256, 4>((int)H.nl_cfg.size(), 4, D.nl_cfg, D.nl_first, D.nl_count, D.np_src, DT.lr_Wp, fe,
                          D.near_z, side, p->tune.near_wgs, R, sFL, sNZ);
    VFX_HIP(hipGetLastError());
    MARK(Plan::evNear1, side);
    {
      int rc = launch_near_ts(p, fe, V, nrhs, p->tune.near_wgs, side, err);
      if (rc) return rc;
    }
    MARK(Plan::evNear2, side);
  } else {
    if (!H.sy_tgt.empty() || !H.nl_cfg.empty()) MARK(Plan::evNear0, side);
    int rc = launch_near_sym(p, fe, nrhs, p->tune.near_wgs, side, err);
    if (rc) return rc;
    MARK(Plan::evNear1, side);
    if (mixed) {
      // pairs in mixed precision: the low-rank and self products of the
      // fixed-point bf16 (mode 1) or int8 (mode 2) slices (FP64 results, rows
      // of the same buffer)
      rc = H.precision == 2 ? launch_near_f8(p, nrhs, p->tune.near_wgs, side, err)
                            : launch_near_fx(p, nrhs, p->tune.near_wgs, side, err);
      if (rc) return rc;
      MARK(Plan::evNear2, side);
    }
  }
  VFX_HIP(hipGetLastError());
  if (!H.up_grp.empty()) {
    MARK(Plan::evUp0, s);
    const int ng = (int)H.up_grp.size() / 5;
#define VFX_UP(PMV, EX)                                                                                            \
  hipLaunchKernelGGL((k_up<PMV, EX>), dim3(ng, R, (P + 7) / 8), dim3(64), 0, s, P, T.root_size, D.up_grp, D.up_box, D.up_ptr,  \
                     D.up_src, D.up_pos, D.box_level, D.box_cx, D.box_cy, DT.pas_m2m_t, D.mpole, D.up_part, sMP,  \
                     sUP)
    if (P == 21)
      VFX_UP(21, true);
    else if (P == 25)
      VFX_UP(25, true);
    else if (P == 31)
      VFX_UP(31, true);
    else if (P == 41)
      VFX_UP(41, true);
    else if (P <= 32)
      VFX_UP(32, false);
    else
      VFX_UP(64, false);
#undef VFX_UP
    if (!H.up_split.empty())
      hipLaunchKernelGGL(k_up_sum, dim3((int)H.up_split.size() / 3, R), dim3(64), 0, s, P, D.up_split, D.up_part,
                         D.mpole, sUP, sMP);
    MARK(Plan::evUp1, s);
  }
  VFX_HIP(hipGetLastError());
  // M2P for list 3 on the side stream, behind the near field, once the
  // upward pass is done; the side stream then joins the caller's
  if (!one) {
    VFX_HIP(hipEventRecord(p->up_ev, s));
    VFX_HIP(hipStreamWaitEvent(side, p->up_ev, 0));
  }
  if (!H.t3_cfg.empty()) MARK(Plan::evM2p0, side);
  m2p_gemm(n, T.p2l_rows, 2 * P, (int)H.t3_cfg.size(), D.t3_cfg, D.t3_first, D.t3_count, D.p3_src, DT.m2p_gemm,
           (const double*)D.mpole, D.m2p_y, side, R, 2 * sMP, sM3);
  VFX_HIP(hipGetLastError());
  if (!H.t3_cfg.empty()) MARK(Plan::evM2p1, side);
  if (!one) VFX_HIP(hipEventRecord(p->join_ev, side));
  if (H.nlev > 2) {
    if (p2l_caller) {
      int rc = p2l(s);
      if (rc) return rc;
    }
    MARK(Plan::evM2l0, s);
    if (!one && !p2l_caller) VFX_HIP(hipStreamWaitEvent(s, p->p2l_ev, 0));  // list-4 products from the side stream
    const int ng = (int)H.m2l_grp.size() - 1;
    const bool split = (long)ng * nrhs <= kM2LSplitGroups;
    if (ng > 0) {
#define VFX_M2L(PMV)                                                                                             \
  hipLaunchKernelGGL(k_m2l_pairs<PMV>, dim3(ng, R), dim3(64), 0, s, P, T.root_size, D.m2l_grp, D.box_level,      \
                     D.l2_ptr, D.l2_src, D.l2_off, D.l2_tgt, D.l4_ptr, D.l4_src, D.l4_slot, D.leaf_box, T.p2l_rows, \
                     DT.pas_m2l_t, DT.m2l_logd, D.mpole, D.p2l_y, D.local, sMP, sPL)
#define VFX_M2LL(PV)                                                                                             \
  if (split)                                                                                                     \
    VFX_M2LS(PV, true, (PV + 7) / 8);                                                                            \
  else                                                                                                           \
    VFX_M2LS(PV, false, 1)
#define VFX_M2LS(PV, SP, NZ)                                                                                     \
  hipLaunchKernelGGL((k_m2l_lanes<PV, SP>), dim3(ng, R, NZ), dim3(64), 0, s, T.root_size, D.m2l_grp, D.box_level, \
                     D.l2_ptr, D.l2_src, D.l2_off, D.l2_tgt, D.l4_ptr, D.l4_src, D.l4_slot, D.leaf_box, T.p2l_rows, \
                     DT.pas_m2l_t, DT.m2l_logd, D.mpole, D.p2l_y, D.local, sMP, sPL)
      if (P == 21)
        VFX_M2LL(21);
      else if (P == 25)
        VFX_M2LL(25);
      else if (P == 31)
        VFX_M2LL(31);
      else if (P == 41)
        VFX_M2LL(41);
      else if (P <= 32)
        VFX_M2L(32);
      else
        VFX_M2L(64);
#undef VFX_M2L
#undef VFX_M2LL
#undef VFX_M2LS
    }
  }
  VFX_HIP(hipGetLastError());
  MARK(Plan::evM2l1, s);
  // full local expansions of the leaves (downward pass)
  {
    const int ng = (int)H.dn_grp.size() - 1;
#define VFX_DOWN(PMV, EX)                                                                                          \
  hipLaunchKernelGGL((k_down<PMV, EX>), dim3(ng, R, (P + 7) / 8), dim3(64), 0, s, P, T.root_size, D.dn_grp, D.anc_ptr, D.anc,   \
                     D.anc_leaf, D.leaf_box, D.box_level, D.box_cx, D.box_cy, DT.pas_l2l_t, D.local, D.locf, sMP,  \
                     sLF)
    if (P == 21)
      VFX_DOWN(21, true);
    else if (P == 25)
      VFX_DOWN(25, true);
    else if (P == 31)
      VFX_DOWN(31, true);
    else if (P == 41)
      VFX_DOWN(41, true);
    else if (P <= 32)
      VFX_DOWN(32, false);
    else
      VFX_DOWN(64, false);
#undef VFX_DOWN
  }
  VFX_HIP(hipGetLastError());
  MARK(Plan::evDown1, s);
  if (!one) VFX_HIP(hipStreamWaitEvent(s, p->join_ev, 0));  // join
  MARK(Plan::evFar0, s);
  {
    const FarArgs A{L,      P,        T.root_size, H.ts,     D.leaf_box,   D.box_level, DT.t,    D.l3_ptr, D.l3_src,
                    D.l3_slot, D.m2p_y, D.locf,  D.mpole, D.l1_ptr, D.l1_srcbox, D.sy_row, D.ysym, D.y_ptr,
                    D.y_slot, D.near_y, V,       sLF,     sMP,      sYS,         sNY,     sM3,      sFL};
    const bool node = H.ts || mixed;
#define VFX_FAR(KV, LPWV)                                                                              \
  if (node)                                                                                            \
    hipLaunchKernelGGL((k_far<KV, true>), dim3((L + 4 * LPWV - 1) / (4 * LPWV), R), dim3(256), 0, s, A); \
  else                                                                                                 \
    hipLaunchKernelGGL((k_far<KV, false>), dim3((L + 4 * LPWV - 1) / (4 * LPWV), R), dim3(256), 0, s, A)
    switch (T.K) {
      case 4: VFX_FAR(4, 16); break;
      case 8: VFX_FAR(8, 4); break;
      case 12: VFX_FAR(12, 1); break;
      default: VFX_FAR(16, 1); break;
    }
#undef VFX_FAR
  }
  VFX_HIP(hipGetLastError());
  MARK(Plan::evEnd, s);
  if (timed) p->n_timed++;
  return VFX_OK;
}

}  // namespace vfx
