// Near field (list 1) and leaf multipoles from folded leaf data and the
// exterior moments (tables.cpp, build_moments), FP64.
//
// The work is the products of T_c with the leaf data for the 33
// configurations of list 1.  Two exact identities cut it to a third:
//   - outside its leaf the potential of a leaf's K^2 values depends on
//     4E = K^2 - (K-4)^2 moments of them only (112 of 256 at K = 16);
//   - reflected neighbours share one operator per parity block, so the
//     self operator costs K^4/4 multiply-adds per target instead of K^4, the
//     two neighbours across x (or y) E K^2 together, and the four corner
//     neighbours 2E K^2 together.
// All same-level sources of a target are summed in registers and leave as
// one row (in folded form, unfolded by the far-field kernel); only the pairs
// of leaves of different levels (about a tenth of list 1 in the inside of a
// tree, a fifth on small ones) write a row each.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>

#include "vfx_internal.h"

namespace vfx {

namespace {

typedef double sy_d4 __attribute__((ext_vector_type(4)));
typedef double sy_d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ sy_d4 sy_mfma(double a, double b, sy_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <int I, int N, class F>
__device__ __forceinline__ void sy_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    sy_for<I + 1, N>(f);
  }
}

template <int K>
struct Dim {
  static constexpr int n = K * K, H = K / 2, H2 = H * H, SH = H2 / 4;
  static constexpr int E = H2 - (H - 2) * (H - 2), SE = E / 4;  // moments per parity, MFMA steps of them
  static constexpr int EP = moment_stride(E);                   // row of one parity's moments, whole cache lines
  static constexpr int RT = (H2 + 15) / 16, R = 16 * RT;        // row tiles of one folded parity
  static constexpr int KS = SH + 8 * SE;                        // MFMA steps per parity of a target
  static constexpr int NC = (SH + 8) / 9, CS = SH / NC;         // the own leaf's steps in chunks of CS <= 9
  static constexpr int NSEG = NC + 8;                           // chunks, then the neighbours' segments
  static constexpr int MX = CS > SE ? CS : SE;
};

// Exterior moments and multipoles of every leaf that is a source: one
// work-group per 16 leaves, whose values are staged in LDS (a wave's lanes
// then read 16 rows at once, which from memory would be 64 cache lines per
// load); wave q folds parity q (A operand, k = SH (l/16) + s) and forms its
// moments and P2M rows by MFMA against mom_T, read from the L2.  Bound by
// latency: the largest trees give two or three work-groups per CU.
template <int K, int NT>
__global__ void __launch_bounds__(256) k_moments(int nleaf, int P, double root_size, const int* __restrict__ leaves,
                                                 const int* __restrict__ leaf_box, const int* __restrict__ box_level,
                                                 const double* __restrict__ momT, const double* __restrict__ fe,
                                                 double* __restrict__ mom, double* __restrict__ mpole, long sfe,
                                                 long smm, long smp) {
  using D = Dim<K>;
  constexpr int LD = D::n + 2, PC = D::n / 2;  // LDS row, 16-byte pieces of a leaf
  __shared__ __attribute__((aligned(16))) double sF[16 * LD];
  fe += blockIdx.y * sfe;  // right-hand side blockIdx.y
  mom += blockIdx.y * smm;
  mpole += blockIdx.y * smp;
  const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int e0 = 16 * blockIdx.x, np = min(16, nleaf - e0);
  const int leaf = leaves[e0 + (li < np ? li : 0)];
#pragma unroll
  for (int v = threadIdx.x; v < 16 * PC; v += 256) {
    const int row = v / PC, pc = v - row * PC;
    const int lr = __shfl(leaf, row, 64);
    *(sy_d2*)(sF + row * LD + 2 * pc) = *(const sy_d2*)(fe + (size_t)lr * D::n + 2 * pc);
  }
  __syncthreads();
  const double* f = sF + li * LD;
  const double sx = (q & 2) ? -1.0 : 1.0, sy = (q & 1) ? -1.0 : 1.0, sxy = sx * sy;
  const double* B = momT + (size_t)q * D::H2 * (16 * NT) + lk * (16 * NT) + li;
  sy_d4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = sy_d4{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < D::SH; ++s) {
    const int k = D::SH * lk + s, ka = k / D::H, kb = k % D::H;
    const double* r0 = f + ka * K;
    const double* r1 = f + (K - 1 - ka) * K;
    const double a = (r0[kb] + sy * r0[K - 1 - kb]) + (sx * r1[kb] + sxy * r1[K - 1 - kb]);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = sy_mfma(a, B[(size_t)s * 4 * (16 * NT) + 16 * t], acc[t]);
  }
  // outputs D[lk + 4e][16 t + li]: leaf e0 + lk + 4e, row 16 t + li
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int en = lk + 4 * e;
    const int lo = __shfl(leaf, en, 64);
    if (en >= np) continue;
    const int b = leaf_box[lo];
    const double h = ldexp(root_size, -box_level[b]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int row = 16 * t + li;
      if (row < D::E) {
        mom[((size_t)lo * 4 + q) * D::EP + row] = acc[t][e];
      } else {
        const int l = 2 * (row - D::E) + ((q == 1 || q == 2) ? 1 : 0);
        if (l < P) mpole[2 * ((size_t)b * P + l) + (q & 1)] = h * h * acc[t][e];
      }
    }
  }
}

// Segments of a target's contraction for parity q = 2 qx + qy: the own leaf's
// folded values in NC chunks, then the moments of the neighbours (nb: own,
// +x, -x, +y, -y, ++, -+, +-, --; a missing one is the zero row, a missing
// own leaf -1), reflected neighbours combined with the signs of their parity.
template <int K, int SG>
struct Seg {
  using D = Dim<K>;
  static constexpr bool own = SG < D::NC;
  static constexpr int g = SG - D::NC;  // 0, 1 x edges; 2, 3 y edges; 4..7 corners
  static constexpr int steps = own ? D::CS : D::SE;
  static constexpr int step0 = own ? SG * D::CS : D::SH + g * D::SE;
  static constexpr int nsrc = own ? 4 : (g < 4 ? 2 : 4);
  static constexpr int first = g < 2 ? 1 : (g < 4 ? 3 : 5);  // first neighbour

  // parity of the source moments, and the signs of the reflected sources
  __device__ __forceinline__ static int par(int q) {
    return g < 2 ? 2 * g + (q & 1) : (g < 4 ? 2 * (q >> 1) + (g - 2) : g - 4);
  }
  __device__ __forceinline__ static double sign(int q, int bit) {  // bit 2: x, 1: y
    return ((own ? q : q ^ par(q)) & bit) ? -1.0 : 1.0;
  }
  // value of the operand from its nsrc source values
  __device__ __forceinline__ static double combine(const double* v, int q) {
    if constexpr (own) {  // images (a,b), (a,b'), (a',b), (a',b')
      return (v[0] + sign(q, 1) * v[1]) + sign(q, 2) * (v[2] + sign(q, 1) * v[3]);
    } else if constexpr (nsrc == 2) {
      return v[0] + sign(q, g < 2 ? 2 : 1) * v[1];
    } else {
      return (v[0] + sign(q, 2) * v[1]) + sign(q, 1) * (v[2] + sign(q, 2) * v[3]);
    }
  }
};

// The lists of both item kinds: same-level targets (nb: nine leaf rows per
// target) and tiles of coarse / fine pairs of one configuration.
struct SymArgs {
  int ntgt;
  const int* nb;
  const double* symT;
  int npair_tiles;
  const int *cfg, *first, *count, *src;
  const double* pairT;
  const double *fe, *mom;
  double *ysym, *ypair;
  long sfe, smm, sys, syp;
};

// K = 16.  Same-level item: 16 TG targets and one parity, whose 64 rows are
// four MFMA row tiles; wave w takes targets 16 (w % TG) .. + 15 and TG of
// the row tiles.  Pair item: 16 TG pairs of one configuration times 64 of the
// 256 target rows, four segments (the source's four parities).  Per segment
// (7 or 8 steps) both operands go through double-buffered LDS, loaded one
// segment ahead of their use:
//   A  the combined source values, 16-byte pieces of whole rows (224 or 256
//      contiguous bytes), so that a load touches a dozen cache lines; read
//      straight into the MFMA's lanes every load would touch 32 to 64, and
//      that, not the matrix cores, bounded the kernel (14254 leaves: 93 us against 62;
//      matrix cores busy 45% of it, 58% in a batch of 32);
//   B  the table block, 28 or 32 rows of 64.
// LDS rows: A 34 doubles (the 32 lanes of a half-wave read 32 different
// pairs of banks in the moment segments, seven steps apart; in the two own-leaf
// chunks, eight apart, two lanes share a pair), B 64 doubles with the tiles of
// odd lane groups swapped in pairs.  Items of one tile of targets are consecutive and every XCD walks a
// contiguous share of the targets and then of the pairs, so its L2 serves the
// neighbours' moments.
constexpr int kSyLDA = 34;

// 16 bytes at base + 16 off (one 64-bit shift-add per address)
__device__ __forceinline__ sy_d2 ld16(const double* base, unsigned off) {
  return *(const sy_d2*)((const char*)base + ((size_t)off << 4));
}

template <int TG, bool PAIR>
__device__ __forceinline__ void sym_item(const SymArgs& S, int item, double* sA, double* sB, unsigned* sN) {
  using D = Dim<16>;
  constexpr int NSEG = PAIR ? 4 : D::NSEG, TE = 16 * TG;
  constexpr int BUFA = TE * kSyLDA, BUFB = 4 * D::MX * 64;
  constexpr int PM = 2 * D::SE, PO = 2 * D::CS;  // 16-byte pieces of a moment row, of an own-leaf chunk
  constexpr int NM = (TE * PM + 255) / 256, NO = (TE * PO + 255) / 256;  // pieces per thread
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int grp = w % TG, wr = w / TG;  // target group and first row tile share
  int p0, np;
  const int tile = item >> 2, q = item & 3;  // q: parity, or the block of 64 target rows
  const double* tab;
  if constexpr (PAIR) {
    constexpr int sub = 4 / TG;  // list tiles hold 64 pairs
    const int lt = tile / sub, off = TE * (tile % sub);
    p0 = S.first[lt] + off;
    np = min(TE, S.count[lt] - off);
    if (np <= 0) return;  // uniform over the work-group
    tab = S.pairT + (size_t)(S.cfg[lt] - 9) * 4 * D::E * D::n + 64 * q;
  } else {
    p0 = TE * tile;
    np = min(TE, S.ntgt - p0);
    tab = S.symT + (size_t)q * D::KS * 4 * D::R;
  }
  constexpr int ldt = PAIR ? D::n : D::R;  // row stride of the table
  __syncthreads();  // the previous item is done with the LDS buffers
  // source rows in 16-byte units: moments EP/2 per parity, leaf values n/2
  if constexpr (PAIR) {
    if (tid < TE) sN[tid] = S.src[p0 + (tid < np ? tid : 0)] * (2u * D::EP);
  } else {
    for (int v = tid; v < 9 * TE; v += 256) {
      const int r = v / 9, u = v - 9 * r;
      const int lf = S.nb[9 * (size_t)(p0 + (r < np ? r : 0)) + u];
      sN[v] = u == 0 ? (lf < 0 ? ~0u : lf * (unsigned)(D::n / 2)) : lf * (2u * D::EP);
    }
  }
  __syncthreads();
  // this thread's moment pieces: operand row and piece of the row, the same
  // in every segment
  int mN[NM], mA[NM];
  unsigned mP[NM];
#pragma unroll
  for (int e = 0; e < NM; ++e) {
    const int v = tid + 256 * e, row = v / PM, pc = v - row * PM;
    mN[e] = PAIR ? row : 9 * row;
    mA[e] = row * kSyLDA + 2 * pc;
    mP[e] = pc;
  }
  sy_d2 ra[NO > NM ? NO : NM][4], rb[4];
  auto load = [&](auto sgc) __attribute__((always_inline)) {
    constexpr int sg = decltype(sgc)::value;
    using SG = Seg<16, PAIR ? 2 : sg>;
    constexpr int steps = PAIR ? D::SE : SG::steps;
    if constexpr (!PAIR && SG::own) {
      // operand l * 16 + 8 sg + s in piece 4 l + s/2: node (a, b), four images
      sy_for<0, NO>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        const int v = tid + 256 * e, row = v / PO, pc = v % PO;
        if (256 * (e + 1) <= TE * PO || v < TE * PO) {
          const unsigned lf = sN[9 * row];
          const unsigned a = 2 * (pc >> 2) + sg, b = pc & 3;
          const sy_d2 z = {0.0, 0.0};
          const unsigned o = lf == ~0u ? 0u : lf;
          ra[e][0] = ld16(S.fe, o + 8 * a + b);
          ra[e][1] = ld16(S.fe, o + 8 * a + 7 - b);
          ra[e][2] = ld16(S.fe, o + 8 * (15 - a) + b);
          ra[e][3] = ld16(S.fe, o + 8 * (15 - a) + 7 - b);
          if (lf == ~0u) ra[e][0] = ra[e][1] = ra[e][2] = ra[e][3] = z;
        }
      });
    } else {
      const unsigned par = (PAIR ? sg : SG::par(q)) * (D::EP / 2);
      sy_for<0, NM>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        if (256 * (e + 1) <= TE * PM || tid + 256 * e < TE * PM) {
#pragma unroll
          for (int u = 0; u < (PAIR ? 1 : SG::nsrc); ++u)
            ra[e][u] = ld16(S.mom, sN[mN[e] + (PAIR ? 0 : SG::first + u)] + mP[e] + par);
        }
      });
    }
    constexpr int pieces = 128 * steps, r0 = 4 * (PAIR ? D::SE * sg : SG::step0);
    sy_for<0, 4>([&](auto ec) __attribute__((always_inline)) {
      constexpr int e = decltype(ec)::value;
      const unsigned v = tid + 256 * e, row = v >> 5, pc = v & 31;
      if (256 * (e + 1) <= pieces || (int)v < pieces) rb[e] = ld16(tab + (size_t)r0 * ldt, row * (ldt / 2) + pc);
    });
  };
  auto store = [&](auto sgc) __attribute__((always_inline)) {
    constexpr int sg = decltype(sgc)::value;
    using SG = Seg<16, PAIR ? 2 : sg>;
    constexpr int steps = PAIR ? D::SE : SG::steps;
    if constexpr (!PAIR && SG::own) {
      sy_for<0, NO>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        const int v = tid + 256 * e, row = v / PO, pc = v % PO;
        if (256 * (e + 1) <= TE * PO || v < TE * PO) {  // the images in y hold the pair in reverse
          const double x[4] = {ra[e][0].x, ra[e][1].y, ra[e][2].x, ra[e][3].y};
          const double y[4] = {ra[e][0].y, ra[e][1].x, ra[e][2].y, ra[e][3].x};
          *(sy_d2*)(sA + (sg & 1) * BUFA + row * kSyLDA + 2 * pc) = sy_d2{SG::combine(x, q), SG::combine(y, q)};
        }
      });
    } else {
      sy_for<0, NM>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = decltype(ec)::value;
        if (256 * (e + 1) <= TE * PM || tid + 256 * e < TE * PM) {
          sy_d2 o = ra[e][0];
          if constexpr (!PAIR) {
            const double x[4] = {ra[e][0].x, ra[e][1].x, ra[e][2].x, ra[e][3].x};
            const double y[4] = {ra[e][0].y, ra[e][1].y, ra[e][2].y, ra[e][3].y};
            o = sy_d2{SG::combine(x, q), SG::combine(y, q)};
          }
          *(sy_d2*)(sA + (sg & 1) * BUFA + mA[e]) = o;
        }
      });
    }
    constexpr int pieces = 128 * steps;
    sy_for<0, 4>([&](auto ec) __attribute__((always_inline)) {
      constexpr int e = decltype(ec)::value;
      const int v = tid + 256 * e, row = v >> 5, col = 2 * (v & 31);
      if (256 * (e + 1) <= pieces || v < pieces)
        *(sy_d2*)(sB + (sg & 1) * BUFB + row * 64 + (col ^ ((row & 1) << 4))) = rb[e];
    });
  };
  sy_d4 acc[TG];
#pragma unroll
  for (int r = 0; r < TG; ++r) acc[r] = sy_d4{0, 0, 0, 0};
  using I0 = std::integral_constant<int, 0>;
  load(I0{});
  store(I0{});
  __syncthreads();
  const double* pa = sA + (16 * grp + li) * kSyLDA;
  const double* pb = sB + lk * 64 + li + 16 * (lk & 1);
  const int flip = 32 * (lk & 1);  // tile r of an odd lane group sits at r ^ 1
  sy_for<0, NSEG>([&](auto sgc) __attribute__((always_inline)) {
    constexpr int sg = decltype(sgc)::value;
    constexpr int ns = PAIR ? D::SE : Seg<16, PAIR ? 2 : sg>::steps;
    using Next = std::integral_constant<int, (sg + 1 < NSEG) ? sg + 1 : 0>;
    if constexpr (sg + 1 < NSEG) load(Next{});
    const double* a0 = pa + (sg & 1) * BUFA + ns * lk;
    const double* b0 = pb + (sg & 1) * BUFB;
#pragma unroll
    for (int s = 0; s < ns; ++s) {
      const double a = a0[s];
#pragma unroll
      for (int r = 0; r < TG; ++r) {
        const int t = TG * wr + r;
        acc[r] = sy_mfma(a, b0[4 * s * 64 + 16 * t - ((t & 1) ? flip : 0)], acc[r]);
      }
    }
    if constexpr (sg + 1 < NSEG) {
      store(Next{});
      __syncthreads();
    }
  });
  // outputs D[lk + 4e][16 r + li]
  double* Y = (PAIR ? S.ypair : S.ysym) + (size_t)p0 * D::n + 64 * q + 16 * TG * wr + li;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int en = 16 * grp + lk + 4 * e;
    if (en >= np) continue;
#pragma unroll
    for (int r = 0; r < TG; ++r) Y[(size_t)en * D::n + 16 * r] = acc[r][e];
  }
}

template <int TG>
__global__ void __launch_bounds__(256, 2) k_near_sym(SymArgs S) {
  using D = Dim<16>;
  __shared__ __attribute__((aligned(16))) double sA[2 * 16 * TG * kSyLDA];
  __shared__ __attribute__((aligned(16))) double sB[2 * 4 * D::MX * 64];
  __shared__ unsigned sN[9 * 16 * TG];
  const long r = blockIdx.y;  // right-hand side
  S.fe += r * S.sfe;
  S.mom += r * S.smm;
  S.ysym += r * S.sys;
  S.ypair += r * S.syp;
  const int nA = 4 * ((S.ntgt + 16 * TG - 1) / (16 * TG)), nB = 4 * (4 / TG) * S.npair_tiles;
  const int nb = gridDim.x, bb = blockIdx.x, x = bb & 7, xwgs = (nb - x + 7) >> 3;
  const int qa = nA >> 3, ra = nA & 7, qb = nB >> 3, rb = nB & 7;
  const int firstA = x * qa + min(x, ra), countA = qa + (x < ra ? 1 : 0);
  const int firstB = x * qb + min(x, rb), countB = qb + (x < rb ? 1 : 0);
  for (int j = bb >> 3; j < countA + countB; j += xwgs) {
    if (j < countA)
      sym_item<TG, false>(S, firstA + j, sA, sB, sN);
    else
      sym_item<TG, true>(S, firstB + j - countA, sA, sB, sN);
  }
}

// np <= 16 sources (src) of one configuration: Y[entry][row] = sum over the
// 4E moments, 16 NRT rows dealt to the four waves (w) in tiles; the sources'
// moments (whole rows) are staged in LDS, the table (steps x 4 x rows) is
// read straight from the L2.
template <int K>
constexpr int kMomLD = 4 * Dim<K>::E + 2;

template <int K, int NRT>
__device__ __forceinline__ void mom_apply(const double* __restrict__ tab, const double* __restrict__ mom,
                                          const int* __restrict__ src, int np, double* __restrict__ Y, int w,
                                          double* sM) {
  using D = Dim<K>;
  constexpr int NT = (NRT + 3) / 4, R = 16 * NRT, PC = 2 * D::E;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  for (int v = threadIdx.x; v < 16 * PC; v += 256) {
    const int row = v / PC, pc = v - row * PC, p = pc / (D::E / 2), c = pc - p * (D::E / 2);
    *(sy_d2*)(sM + row * kMomLD<K> + 2 * pc) =
        *(const sy_d2*)(mom + ((size_t)src[row < np ? row : 0] * 4 + p) * D::EP + 2 * c);
  }
  __syncthreads();
  const double* m = sM + li * kMomLD<K> + D::SE * lk;
  tab += lk * R + li;
  sy_d4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = sy_d4{0, 0, 0, 0};
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int s = 0; s < D::SE; ++s) {
      const double a = m[p * D::E + s];
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = sy_mfma(a, tab[(size_t)(D::SE * p + s) * 4 * R + 16 * min(w + 4 * t, NRT - 1)], acc[t]);
    }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int en = lk + 4 * e;
    if (en >= np) continue;
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (w + 4 * t < NRT) Y[(size_t)en * R + 16 * (w + 4 * t) + li] = acc[t][e];
  }
}

// K < 16, whose tables fit an XCD's L2 many times over: no shared table
// blocks, the table operands come straight from the L2.  Same-level: 16
// targets per work-group, wave q forms parity q (its row tiles); operands are
// loaded one segment ahead.  Pairs: 16 pairs of a configuration, the K^2/16
// row tiles dealt to the four waves.
template <int K>
__global__ void __launch_bounds__(256) k_near_sym_small(SymArgs S, int nA) {
  using D = Dim<K>;
  __shared__ __attribute__((aligned(16))) double sM[16 * kMomLD<K>];
  const long rr = blockIdx.y;  // right-hand side
  S.fe += rr * S.sfe;
  S.mom += rr * S.smm;
  S.ysym += rr * S.sys;
  S.ypair += rr * S.syp;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  if ((int)blockIdx.x < nA) {
    constexpr int NT = D::RT;
    const int q = w;
    const int p0 = 16 * blockIdx.x, np = min(16, S.ntgt - p0);
    int nb[9];
#pragma unroll
    for (int u = 0; u < 9; ++u) nb[u] = S.nb[9 * (size_t)(p0 + (li < np ? li : 0)) + u];
    const double* tab = S.symT + ((size_t)q * D::KS * 4 + lk) * D::R + li;
    double raw[4][D::MX], a[D::MX], bn[NT][D::MX], b[NT][D::MX];
    sy_d4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = sy_d4{0, 0, 0, 0};
    auto load = [&](auto sgc) __attribute__((always_inline)) {
      using SG = Seg<K, decltype(sgc)::value>;
#pragma unroll
      for (int s = 0; s < SG::steps; ++s) {
        if constexpr (SG::own) {
          const int k = D::SH * lk + D::CS * decltype(sgc)::value + s, ka = k / D::H, kb = k % D::H;
          const double* f = S.fe + (size_t)max(nb[0], 0) * D::n;
          raw[0][s] = nb[0] < 0 ? 0.0 : f[ka * K + kb];
          raw[1][s] = nb[0] < 0 ? 0.0 : f[ka * K + K - 1 - kb];
          raw[2][s] = nb[0] < 0 ? 0.0 : f[(K - 1 - ka) * K + kb];
          raw[3][s] = nb[0] < 0 ? 0.0 : f[(K - 1 - ka) * K + K - 1 - kb];
        } else {
#pragma unroll
          for (int u = 0; u < SG::nsrc; ++u)
            raw[u][s] = S.mom[((size_t)nb[SG::first + u] * 4 + SG::par(q)) * D::EP + D::SE * lk + s];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) bn[t][s] = tab[(size_t)(SG::step0 + s) * 4 * D::R + 16 * t];
      }
    };
    load(std::integral_constant<int, 0>{});
    sy_for<0, D::NSEG>([&](auto sgc) __attribute__((always_inline)) {
      constexpr int sg = decltype(sgc)::value;
      using SG = Seg<K, sg>;
#pragma unroll
      for (int s = 0; s < SG::steps; ++s) {
        const double v[4] = {raw[0][s], raw[1][s], SG::nsrc == 4 ? raw[2][s] : 0.0, SG::nsrc == 4 ? raw[3][s] : 0.0};
        a[s] = SG::combine(v, q);
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t][s] = bn[t][s];
      }
      if constexpr (sg + 1 < D::NSEG) load(std::integral_constant<int, sg + 1>{});
#pragma unroll
      for (int s = 0; s < SG::steps; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = sy_mfma(a[s], b[t][s], acc[t]);
    });
    double* Y = S.ysym + (size_t)p0 * D::n + q * D::H2;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int en = lk + 4 * e;
      if (en >= np) continue;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int row = 16 * t + li;
        if (row < D::H2) Y[(size_t)en * D::n + row] = acc[t][e];
      }
    }
    return;
  }
  // pairs: tiles of <= 64 of one configuration, four work-groups per tile
  const int item = blockIdx.x - nA, tile = item >> 2, sub = 16 * (item & 3);
  const int p0 = S.first[tile] + sub, np = min(16, S.count[tile] - sub);
  if (np > 0)
    mom_apply<K, D::n / 16>(S.pairT + (size_t)(S.cfg[tile] - 9) * 4 * D::E * D::n, S.mom, S.src + p0, np,
                            S.ypair + (size_t)p0 * D::n, w, sM);
}

// P2L (list 4): the local expansion's 2(p+1) real rows (padded to 16 NRT)
// from the source's moments, one row per entry; tiles as for the pairs.
template <int K, int NRT>
__global__ void __launch_bounds__(256) k_p2l(const int* __restrict__ cfg, const int* __restrict__ first,
                                             const int* __restrict__ count, const int* __restrict__ src,
                                             const double* __restrict__ tab, const double* __restrict__ mom,
                                             double* __restrict__ Y, long smm, long sy) {
  __shared__ __attribute__((aligned(16))) double sM[16 * kMomLD<K>];
  const int tile = blockIdx.x >> 2, sub = 16 * (blockIdx.x & 3);
  const int p0 = first[tile] + sub, np = min(16, count[tile] - sub);
  if (np > 0)
    mom_apply<K, NRT>(tab + (size_t)cfg[tile] * 4 * Dim<K>::E * (16 * NRT), mom + blockIdx.y * smm, src + p0, np,
                      Y + blockIdx.y * sy + (size_t)p0 * (16 * NRT), __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                      sM);
}

template <int K>
void moments(const Plan* p, const double* fe, int nrhs, hipStream_t s) {
  const HostPlan& H = p->H;
  const DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  const int nl = (int)H.leaf_ids.size(), P = T.p + 1;
  const long rows = H.L + 1;  // and the zero row
#define VFX_MOM(NTV)                                                                                               \
  case NTV:                                                                                                        \
    hipLaunchKernelGGL((k_moments<K, NTV>), dim3((nl + 15) / 16, nrhs), dim3(256), 0, s, nl, P, T.root_size,       \
                       D.leaf_ids, D.leaf_box, D.box_level, p->ctx->D.mom_T, fe, D.mom, (double*)D.mpole,          \
                       (long)H.L * T.n, rows * 4 * moment_stride(T.mom_E), 2L * H.B * P);                                         \
    break;
  switch (T.mom_rows / 16) { VFX_MOM(1) VFX_MOM(2) VFX_MOM(3) VFX_MOM(4) }
#undef VFX_MOM
}

template <int K>
void p2l(const Plan* p, int nrhs, hipStream_t s) {
  const HostPlan& H = p->H;
  const DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  const dim3 grid(4 * (unsigned)H.t4_cfg.size(), nrhs);
  const long smm = (long)(H.L + 1) * 4 * moment_stride(T.mom_E), sy = (long)H.p4_src.size() * T.p2l_rows;
  if (T.p2l_rows == 64)
    hipLaunchKernelGGL((k_p2l<K, 4>), grid, dim3(256), 0, s, D.t4_cfg, D.t4_first, D.t4_count, D.p4_src,
                       p->ctx->D.p2l_gemm, D.mom, D.p2l_y, smm, sy);
  else
    hipLaunchKernelGGL((k_p2l<K, 8>), grid, dim3(256), 0, s, D.t4_cfg, D.t4_first, D.t4_count, D.p4_src,
                       p->ctx->D.p2l_gemm, D.mom, D.p2l_y, smm, sy);
}

}  // namespace

int launch_p2l(const Plan* p, int nrhs, hipStream_t s, std::string& err) {
  if (p->H.t4_cfg.empty()) return VFX_OK;
  switch (p->ctx->T.K) {
    case 4: p2l<4>(p, nrhs, s); break;
    case 8: p2l<8>(p, nrhs, s); break;
    case 12: p2l<12>(p, nrhs, s); break;
    default: p2l<16>(p, nrhs, s); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    err = std::string("p2l: ") + hipGetErrorString(e);
    return VFX_EHIP;
  }
  return VFX_OK;
}

// Exterior moments and multipoles of every leaf with possibly nonzero data.
int launch_moments(const Plan* p, const double* fe, int nrhs, hipStream_t s, std::string& err) {
  if (p->H.leaf_ids.empty()) return VFX_OK;
  switch (p->ctx->T.K) {
    case 4: moments<4>(p, fe, nrhs, s); break;
    case 8: moments<8>(p, fe, nrhs, s); break;
    case 12: moments<12>(p, fe, nrhs, s); break;
    default: moments<16>(p, fe, nrhs, s); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    err = std::string("moments: ") + hipGetErrorString(e);
    return VFX_EHIP;
  }
  return VFX_OK;
}

// List 1 in FP64: same-level pairs (one folded row per target) and the pairs
// of leaves of different levels (one row each).
int launch_near_sym(const Plan* p, const double* fe, int nrhs, int max_wgs, hipStream_t s, std::string& err) {
  const HostPlan& H = p->H;
  const DevicePlan& D = p->D;
  const Tables& T = p->ctx->T;
  const DeviceTables& DT = p->ctx->D;
  const int ntgt = (int)H.sy_tgt.size(), npt = (int)H.nl_cfg.size();
  if (ntgt + npt == 0) return VFX_OK;
  const SymArgs S{ntgt,   D.sy_nb, DT.sym_T, npt,      D.nl_cfg,        D.nl_first,
                  D.nl_count, D.np_src, DT.pair_T, fe, D.mom, D.ysym, D.near_y, (long)H.L * T.n,
                  (long)(H.L + 1) * 4 * moment_stride(T.mom_E), (long)ntgt * T.n, (long)H.np_src.size() * T.n};
  if (T.K == 16) {
    // targets per item: as many as leave every CU a few items
    auto items = [&](int tg) { return 4 * ((ntgt + 16 * tg - 1) / (16 * tg) + (4 / tg) * npt); };
    auto grid = [&](int n) { return std::max((max_wgs > 0 && n > max_wgs) ? max_wgs : n, std::min(n, 8)); };
    if ((long)items(4) * nrhs >= kSymItems4)
      hipLaunchKernelGGL(k_near_sym<4>, dim3(grid(items(4)), nrhs), dim3(256), 0, s, S);
    else if ((long)items(2) * nrhs >= kSymItems2)
      hipLaunchKernelGGL(k_near_sym<2>, dim3(grid(items(2)), nrhs), dim3(256), 0, s, S);
    else
      hipLaunchKernelGGL(k_near_sym<1>, dim3(grid(items(1)), nrhs), dim3(256), 0, s, S);
  } else {
    const int nA = (ntgt + 15) / 16;
    const dim3 g(nA + 4 * npt, nrhs);
    switch (T.K) {
      case 4: hipLaunchKernelGGL(k_near_sym_small<4>, g, dim3(256), 0, s, S, nA); break;
      case 8: hipLaunchKernelGGL(k_near_sym_small<8>, g, dim3(256), 0, s, S, nA); break;
      default: hipLaunchKernelGGL(k_near_sym_small<12>, g, dim3(256), 0, s, S, nA); break;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    err = std::string("near field: ") + hipGetErrorString(e);
    return VFX_EHIP;
  }
  return VFX_OK;
}

}  // namespace vfx
