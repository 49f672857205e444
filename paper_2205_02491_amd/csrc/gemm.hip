// Tile GEMM on CDNA4 matrix cores (MFMA) for complex and real data, with the
// epilogues the ChASE hot path needs fused in:
//   - the Chebyshev step of Eq. (3): out = alpha*(H X_s - gamma X_s) + beta X_{s-2}
//     (the shift of H by gamma is applied to the product, so H stays const),
//     optionally + c_j F_j (the forcing term of the filter's defect form),
//   - split-K partial sums for the tall-skinny Gram / projection products of
//     the QR and Rayleigh-Ritz steps,
//   - per-column residual norms ||H v - lambda v||^2 of the residual step,
//   - the shifted product H P - P diag(lambda) of the eigenvector adjoint.
//
// Operands go from memory straight into MFMA fragments: every wave owns FM x
// FN fragments of 16 x 16 of C and loads its own operand fragments S stages
// ahead of the matrix instructions that use them, 16 bytes a lane.  There is
// no LDS staging and no barrier in the K loop, so waves never wait for one
// another.  An FP64 MFMA occupies the matrix core for 64 cycles; a wave of 3 x
// 2 complex fragments needs 5 loads per 18 of them, which the vector caches
// deliver beside the arithmetic.
//
// The WK waves of a workgroup share one tile of C and deal the K range among
// them (units of 128 contiguous bytes); their partial tiles meet in LDS at
// the end.  Small tiles with the K range split inside the workgroup fill the
// chip from blocks of a few columns on, and waste little on ragged edges.  The
// FP32 filter step has a second kernel, staged through LDS, for wide blocks of
// matrices whose columns lie off the cache lines (staged_f32_kernel).
//
// Measured per filter step against the earlier kernel (128 x 64 and 128 x 128
// tiles staged through double-buffered LDS, one K range per tile), complex:
// n=20000, 1300 columns 54.7 -> 46 ms (90 TFLOP/s algorithmic, 86% of the
// three-product FP64 peak); 1000 x 140 220 -> 22 us; 256 x 16 57 -> 5 us; real:
// 5003 x 173 798 -> 157 us.  At full size the clock is power limited: on
// operands with 16-bit mantissas the same kernel reaches 95 TFLOP/s, and what
// moves fewer bytes between the caches is faster (two waves that share their
// B fragments through the vector cache: 83 -> 88).  Two waves per SIMD are
// needed (one: 62-74 TFLOP/s with larger wave tiles), and the wait counters
// must be exact: a prologue of conditional loads made the compiler wait for
// every load in flight at the head of the loop and cost 5%.
//
// A complex product is three real MFMAs (Gauss: re*re, im*im,
// (re+im)*(re+im)) in the filter and the other long products, four
// (re*re, -im*im, re*im, im*re) in the short products of QR/Rayleigh-Ritz.
// The MFMA is issued with the B fragment in the "A" slot so that each lane's
// four accumulator values lie along a row of C (one column each): the 16
// lanes of a group then write 16 consecutive rows of a column-major output.
// Workgroup ids are remapped so that each of the 8 XCDs (private L2) works on
// a contiguous range of tiles, i.e. on the same few row panels of A.
#include "common.h"

#include <algorithm>

namespace chase {
namespace {

constexpr int NCU = 256;  // compute units of the MI355X

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));

// Element as stored in memory (complex: an interleaved pair).
template <typename TM, bool CPLX>
struct El {
  using type = TM;
};
template <>
struct El<double, true> {
  using type = d2v;
};
template <>
struct El<float, true> {
  using type = f2v;
};

__device__ __forceinline__ double re_(double x) { return x; }
__device__ __forceinline__ double re_(d2v x) { return x.x; }
__device__ __forceinline__ double im_(double) { return 0.0; }
__device__ __forceinline__ double im_(d2v x) { return x.y; }

template <typename TC>
struct MF;
template <>
struct MF<double> {
  using acc_t = d4;
  __device__ static __forceinline__ acc_t fma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct MF<float> {
  using acc_t = f4;
  __device__ static __forceinline__ acc_t fma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Column (within a 16 x 16 fragment of C) of accumulator register r in lane
// group lk = lane/16.  With the operands swapped (B fragment first) the
// fragment is C^T: the FP32 16x16x4 MFMA puts register r of lane group lk
// at row 4*lk + r of its result, the FP64 one at row lk + 4*r.
template <typename TC>
__device__ constexpr int frag_col(int lk, int r) {
  return sizeof(TC) == 8 ? lk + 4 * r : 4 * lk + r;
}

// Fragments of one operand for one pipeline stage: K steps of 4 times KSUB
// (complex: 1, real: 2), so that every load is 16 bytes.  KC: the operand is
// contiguous along K (A^H as stored K x M, B as stored K x N).  F fragments
// along the tile's dimension.
//   complex:          lane (l16, lk) holds element (f 16 + l16, k = lk)
//   real, KC:         lane holds k = 2 lk and 2 lk + 1 of index f 16 + l16
//   real, not KC:     lane holds indices 32 p + 2 l16 and + 1 (fragments 2p
//                     and 2p + 1) of k = 2 lk + s, s = 0, 1; for odd F a
//                     single index f 16 + l16
// The order of k within a stage is free as long as A and B agree.
// Indices past the end are clamped: they only reach entries of C that are not
// stored.  A pair is clamped as a whole (`index`), so that the last index of
// an odd range sits in its lane's second half.
template <typename TM, bool CPLX, bool KC, int F>
struct Frag {
  using T = typename El<TM, CPLX>::type;  // an element in memory
  using T2 = typename El<TM, true>::type;
  static constexpr int KSUB = CPLX ? 1 : 2;
  static constexpr bool PAIR = !CPLX && !KC && F % 2 == 0;
  static constexpr int NV = PAIR ? F : (!CPLX && !KC) ? 2 * F : F;  // values held
  using V = typename El<TM, CPLX || PAIR || KC>::type;             // of this type
  typedef T2 T2u __attribute__((aligned(sizeof(TM))));  // two elements, aligned as one
  struct Ptr {
    const T* p[PAIR ? F / 2 : F];
  };
  // first index of the lane for fragment f, without clamping
  __device__ static __forceinline__ int64_t own(int64_t base, int f, int l) {
    return base + (PAIR ? (f >> 1) * 32 + 2 * l : f * 16 + l);
  }
  // index whose data fragment f holds (base: first index of the wave's part)
  __device__ static __forceinline__ int64_t index(int64_t base, int f, int l, int64_t lim) {
    const int64_t i = own(base, f, l);
    if constexpr (PAIR)
      return (i < lim - 1 ? i : lim - 2) + (f & 1);
    else
      return i < lim ? i : lim - 1;
  }
  // whether that entry of C is this lane's to store (a clamped one belongs to
  // another lane)
  __device__ static __forceinline__ bool mine(int64_t base, int f, int l, int64_t lim) {
    const int64_t i = own(base, f, l);
    return PAIR ? index(base, f, l, lim) >= i : i < lim;
  }
  __device__ static __forceinline__ void init(Ptr& q, const T* X, int64_t ld, int64_t base,
                                              int64_t lim, int64_t k, int l16, int lk) {
    k += KSUB * lk;
#pragma unroll
    for (int f = 0; f < (PAIR ? F / 2 : F); ++f) {
      const int64_t i = index(base, PAIR ? 2 * f : f, l16, lim);
      q.p[f] = X + (KC ? k + i * ld : i + k * ld);
    }
  }
  __device__ static __forceinline__ void load(V (&v)[NV], Ptr& q, int64_t ld, int64_t adv) {
#pragma unroll
    for (int f = 0; f < (PAIR ? F / 2 : F); ++f) {
      if constexpr (CPLX) {
        v[f] = *q.p[f];
      } else if constexpr (KC) {
        v[f] = *reinterpret_cast<const T2u*>(q.p[f]);
      } else if constexpr (PAIR) {
        v[2 * f] = *reinterpret_cast<const T2u*>(q.p[f]);
        v[2 * f + 1] = *reinterpret_cast<const T2u*>(q.p[f] + ld);
      } else {
        v[2 * f] = q.p[f][0];
        v[2 * f + 1] = q.p[f][ld];
      }
      q.p[f] += adv;
    }
  }
  // the partial stage: entries k >= krem are zero (their memory belongs to
  // other rows or columns, or to nothing)
  __device__ static __forceinline__ void load_part(V (&v)[NV], const Ptr& q, int64_t ld, int lk,
                                                   int krem) {
    const int k = KSUB * lk;
#pragma unroll
    for (int f = 0; f < NV; ++f) v[f] = V(0);
#pragma unroll
    for (int f = 0; f < (PAIR ? F / 2 : F); ++f) {
      if constexpr (CPLX) {
        if (k < krem) v[f] = *q.p[f];
      } else if constexpr (KC) {
        if (k < krem) v[f].x = q.p[f][0];
        if (k + 1 < krem) v[f].y = q.p[f][1];
      } else if constexpr (PAIR) {
        if (k < krem) v[2 * f] = *reinterpret_cast<const T2u*>(q.p[f]);
        if (k + 1 < krem) v[2 * f + 1] = *reinterpret_cast<const T2u*>(q.p[f] + ld);
      } else {
        if (k < krem) v[2 * f] = q.p[f][0];
        if (k + 1 < krem) v[2 * f + 1] = q.p[f][ld];
      }
    }
  }
  __device__ static __forceinline__ TM re(const V (&v)[NV], int f, int s) {
    if constexpr (CPLX) return v[f].x;
    else if constexpr (KC) return s ? v[f].y : v[f].x;
    else if constexpr (PAIR) return (f & 1) ? v[(f & ~1) + s].y : v[(f & ~1) + s].x;
    else return v[2 * f + s];
  }
  __device__ static __forceinline__ TM im(const V (&v)[NV], int f) {
    if constexpr (CPLX) return v[f].y;
    else return TM(0);
  }
};

template <typename TA, typename TC, bool CPLX, int OPA, int OPB, int EPI, bool G3, int FM, int FN, int WM, int WN, int WK,
          int S, int OCC = 1>
__global__ __launch_bounds__(64 * WM * WN * WK, OCC) void gemm_kernel(GemmArgs g, int tiles_n,
                                                                    int ntiles) {
  using T = typename El<double, CPLX>::type;  // element of B and C
  using acc_t = typename MF<TC>::acc_t;
  constexpr bool GAUSS = CPLX && G3;
  constexpr int NTHR = 64 * WM * WN * WK;
  constexpr int TBM = WM * FM * 16, TBN = WN * FN * 16;

  // XCD-aware tile index: consecutive hardware ids go round-robin over the
  // 8 XCDs; give each XCD a contiguous range of logical tiles.
  const int per_xcd = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= ntiles) return;
  int tm = t / tiles_n, tn = t - tm * tiles_n;
  if constexpr (EPI == EPI_SPLITK) {
    if (g.tri) {
      // the tiles with tm <= tn, column by column: t = tn (tn + 1) / 2 + tm
      int c = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
      if ((c + 1) * (c + 2) / 2 <= t) ++c;
      if (c * (c + 1) / 2 > t) --c;
      tn = c;
      tm = t - c * (c + 1) / 2;
    }
  }
  const int64_t m0 = (int64_t)tm * TBM, n0 = (int64_t)tn * TBN;
  const int64_t M = g.M, N = g.N;
  int64_t kbeg = 0, kend = g.K;
  if constexpr (EPI == EPI_SPLITK) {
    kbeg = (int64_t)blockIdx.z * g.kslice;
    kend = kbeg + g.kslice < g.K ? kbeg + g.kslice : g.K;
  }
  if constexpr (EPI == EPI_STORE && OPB == OP_N) {
    // B upper triangular from row tri_row0: rows past tri_row0 + n0 + TBN
    // of this column tile are zero
    if (g.tri && g.tri_row0 + n0 + TBN < kend) kend = g.tri_row0 + n0 + TBN;
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave / (WM * WN), wmn = wave - wk * (WM * WN);
  const int wm = wmn / WN, wn = wmn - wm * WN;
  const int l16 = lane & 15, lk = lane >> 4;

  // two products in one pass: each of the two waves of a tile takes one of
  // them whole instead of half of the only one
  constexpr bool PAIR = EPI == EPI_STORE && OPB == OP_C && WK == 2;
  const bool pair = PAIR && g.K2 > 0, second = pair && wk == 1;
  if (second) kend = g.K2;

  using TAe = typename El<TA, CPLX>::type;
  const TAe* __restrict__ A = static_cast<const TAe*>(second ? g.A2 : g.A);
  const T* __restrict__ B = static_cast<const T*>(second ? g.B2 : g.B);
  const int64_t lda = second ? g.lda2 : g.lda, ldb = second ? g.ldb2 : g.ldb;

  using FA = Frag<TA, CPLX, OPA == OP_C, FM>;
  using FB = Frag<double, CPLX, OPB == OP_N, FN>;
  constexpr int KSUB = FA::KSUB, KS = 4 * KSUB;  // K entries of a stage

  // Stages of this wave: units of two stages (128 contiguous bytes along K)
  // dealt round-robin to the WK waves that share a tile; nfull full stages,
  // then perhaps the partial one (krem entries).
  const int64_t klen = kend > kbeg ? kend - kbeg : 0;
  const int64_t stages = klen / KS;
  int64_t nfull;
  {
    const int64_t un = stages >> 1;  // whole units
    nfull = 2 * (un / WK + (wk < (int)(un % WK) ? 1 : 0));
    if ((stages & 1) && (int)(un % WK) == wk) nfull += 1;
    if (pair) nfull = stages;
  }
  const int krem = (int)(klen % KS);
  // the partial stage belongs to the wave whose turn it is
  const bool has_rem = krem != 0 && (pair || (int)((stages >> 1) % WK) == wk);

  const int64_t mw = m0 + wm * FM * 16, nw = n0 + wn * FN * 16;  // this wave's part of C
  typename FA::Ptr pa;
  typename FB::Ptr pb;
  const int64_t kfirst = pair ? 0 : kbeg + 2 * KS * (int64_t)wk;
  FA::init(pa, A, lda, mw, M, kfirst, l16, lk);
  FB::init(pb, B, ldb, nw, N, kfirst, l16, lk);
  // pointer advance after the first / second stage of a unit
  constexpr int64_t adv0 = KS;
  const int64_t adv1 = pair ? KS : (2 * WK - 1) * KS;
  const int64_t a0 = OPA == OP_N ? adv0 * lda : adv0, a1 = OPA == OP_N ? adv1 * lda : adv1;
  const int64_t b0 = OPB == OP_N ? adv0 : adv0 * ldb, b1 = OPB == OP_N ? adv1 : adv1 * ldb;

  // The partial tiles are finished a column fragment at a time: ENT entries,
  // dealt to the threads.  The real rank-k updates, short in K and bound by C,
  // read their entries of C before the K loop: read where they are used, behind
  // the bounds of each entry, they came one memory latency after another (order
  // 20000, rank 1: 1.94 -> 1.36 ms, 4.7 TB/s).
  constexpr int ROWS = TBM, COLS = WN * 16, ENT = ROWS * COLS;
  constexpr bool AHEAD = EPI == EPI_STORE && OPB == OP_C && !CPLX && WK == 2 && FM * FN == 4;
  double* __restrict__ Cd = static_cast<double*>(g.C);
  T yc[AHEAD ? FN : 1][AHEAD ? ENT / NTHR : 1];
  if constexpr (AHEAD) {
    static_assert(ENT % NTHR == 0, "whole rounds of the threads");
    if (g.beta != 0.0)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int u = 0; u < ENT / NTHR; ++u) {
          const int e = threadIdx.x + u * NTHR, c = e / ROWS;
          const int64_t i = m0 + e % ROWS < M ? m0 + e % ROWS : M - 1;
          const int64_t j = FB::index(n0 + (c / 16) * FN * 16, fn, c & 15, N);
          yc[fn][u] = reinterpret_cast<const T*>(Cd)[i + j * g.ldc];
        }
  }

  typename FA::V fa[S][FA::NV];
  typename FB::V fb[S][FB::NV];
  static_assert(S % 2 == 0, "the pipeline covers whole units");
  auto load = [&](int s) {
    FA::load(fa[s], pa, lda, (s & 1) ? a1 : a0);
    FB::load(fb[s], pb, ldb, (s & 1) ? b1 : b0);
  };

  acc_t acc_re[FM][FN], acc_im[CPLX ? FM : 1][CPLX ? FN : 1], acc_s[GAUSS ? FM : 1][GAUSS ? FN : 1];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      acc_re[fm][fn] = acc_t{0, 0, 0, 0};
      if constexpr (CPLX) acc_im[fm][fn] = acc_t{0, 0, 0, 0};
      if constexpr (GAUSS) acc_s[fm][fn] = acc_t{0, 0, 0, 0};
    }

  // C += op(a) op(b) of one K step.  Signs of a conjugated operand go to the
  // B fragments (FN of them).
  auto compute = [&](const typename FA::V (&a)[FA::NV], const typename FB::V (&b)[FB::NV]) {
    if constexpr (GAUSS) {
      TC ar[FM], ai[FM], as[FM], br[FN], bi[FN], bs[FN];
#pragma unroll
      for (int f = 0; f < FM; ++f) {
        ar[f] = (TC)FA::re(a, f, 0);
        ai[f] = (TC)FA::im(a, f);
        as[f] = ar[f] + ai[f];
      }
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        br[f] = (TC)FB::re(b, f, 0);
        bi[f] = (TC)FB::im(b, f);
        bs[f] = br[f] + bi[f];
      }
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
          acc_re[fm][fn] = MF<TC>::fma(br[fn], ar[fm], acc_re[fm][fn]);
          acc_im[fm][fn] = MF<TC>::fma(bi[fn], ai[fm], acc_im[fm][fn]);
          acc_s[fm][fn] = MF<TC>::fma(bs[fn], as[fm], acc_s[fm][fn]);
        }
    } else if constexpr (CPLX) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const TC br = FB::re(b, fn, 0), bi = FB::im(b, fn), nbi = -bi;
        const TC bim = OPB == OP_C ? nbi : bi;     // im of op(b)
        const TC bre_ai = OPA == OP_C ? -br : br;  // factors of a.im as stored
        const TC bim_ai = (OPA == OP_C) != (OPB == OP_C) ? bi : nbi;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
          acc_re[fm][fn] = MF<TC>::fma(br, FA::re(a, fm, 0), acc_re[fm][fn]);
          acc_im[fm][fn] = MF<TC>::fma(bim, FA::re(a, fm, 0), acc_im[fm][fn]);
        }
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
          acc_re[fm][fn] = MF<TC>::fma(bim_ai, FA::im(a, fm), acc_re[fm][fn]);
          acc_im[fm][fn] = MF<TC>::fma(bre_ai, FA::im(a, fm), acc_im[fm][fn]);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < KSUB; ++s)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
            acc_re[fm][fn] = MF<TC>::fma((TC)FB::re(b, fn, s), (TC)FA::re(a, fm, s), acc_re[fm][fn]);
    }
  };

  static_assert(!(GAUSS && (OPA == OP_C || OPB == OP_C)), "three-product form: operands as stored");

  {
    int64_t left = nfull;  // full stages not yet computed
    if (left >= 2 * S) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        load(s);
        __builtin_amdgcn_sched_barrier(0);
      }
      do {
#pragma unroll
        for (int s = 0; s < S; ++s) {
          compute(fa[s], fb[s]);
          load(s);
          __builtin_amdgcn_sched_barrier(0);
        }
        left -= S;
      } while (left >= 2 * S);
    } else {
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (s < left) load(s);
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (s < left) {
        compute(fa[s], fb[s]);
        if (s + S < left) load(s);
      }
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (s + S < left) compute(fa[s], fb[s]);
    if (has_rem) {
      typename FA::V a[FA::NV];
      typename FB::V b[FB::NV];
      FA::load_part(a, pa, lda, lk, krem);
      FB::load_part(b, pb, ldb, lk, krem);
      compute(a, b);
    }
  }

  if constexpr (GAUSS) {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const acc_t p1 = acc_re[fm][fn], p2 = acc_im[fm][fn];
        acc_re[fm][fn] = p1 - p2;
        acc_im[fm][fn] = acc_s[fm][fn] - p1 - p2;
      }
  }

  if constexpr (PAIR) {
    const double f = second ? g.ratio2 : 1.0;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        acc_re[fm][fn] *= f;
        if constexpr (CPLX) acc_im[fm][fn] *= f;
      }
  }

  // ---------------------------------------------------------------- epilogue
  // register r of fragment (fm, fn) holds C's row FA::index(mw, fm, l16) and
  // column FB::index(nw, fn, lk + 4 r)
  auto finish = [&](int64_t i, int64_t j, double vr, double vi, double& colsum, const T* yc) {
    if constexpr (EPI == EPI_RESID || EPI == EPI_SHIFT) {
      const double lam = g.lambda[j];
      const T v = static_cast<const T*>(g.V)[i + j * g.ldv];
      vr -= lam * re_(v);
      if constexpr (CPLX) vi -= lam * im_(v);
      if constexpr (EPI == EPI_RESID) colsum += vr * vr + vi * vi;
      if (EPI == EPI_SHIFT || g.F) {
        if constexpr (CPLX)
          static_cast<T*>(g.F)[i + j * g.ldf] = T{vr, vi};
        else
          static_cast<T*>(g.F)[i + j * g.ldf] = vr;
      }
    } else if constexpr (EPI == EPI_SPLITK) {
      const int64_t o = (int64_t)blockIdx.z * M * N + i + j * M;
      if constexpr (CPLX)
        reinterpret_cast<T*>(Cd)[o] = T{vr, vi};
      else
        Cd[o] = vr;
    } else {
      const int64_t o = i + j * g.ldc;
      if constexpr (EPI == EPI_CHEB) {
        // X_s is the B operand (N form, square H): element (i, j) of B
        const T x = B[i + j * g.ldb];
        vr = g.alpha * (vr - g.gamma * re_(x));
        vi = g.alpha * (vi - g.gamma * im_(x));
      } else {
        vr *= g.alpha;
        vi *= g.alpha;
      }
      if (g.beta != 0.0) {
        const T y = yc ? *yc : reinterpret_cast<const T*>(Cd)[o];
        vr += g.beta * re_(y);
        vi += g.beta * im_(y);
      }
      if constexpr (EPI == EPI_CHEB) {
        if (g.colcoef) {
          const double cj = g.colcoef[j];
          const T f = static_cast<const T*>(g.F)[i + j * g.ldf];
          vr += cj * re_(f);
          vi += cj * im_(f);
        }
      }
      if constexpr (CPLX)
        reinterpret_cast<T*>(Cd)[o] = T{vr, vi};
      else
        Cd[o] = vr;
    }
  };

  if constexpr (WK > 1) {
    // The WK partial tiles meet in LDS, one column fragment at a time; then
    // every thread of the workgroup finishes its share of the entries.
    static_assert(EPI != EPI_RESID || (ROWS <= 64 && (ROWS & (ROWS - 1)) == 0),
                  "a column's rows are a lane group of one wave");
    __shared__ T part[WK][COLS][ROWS];
    __shared__ double csum[EPI == EPI_RESID ? TBN : 1];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      if (fn > 0) __syncthreads();
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        if (!FA::mine(mw, fm, l16, M)) continue;
        const int row = (int)(FA::index(mw, fm, l16, M) - m0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (CPLX)
            part[wk][wn * 16 + frag_col<TC>(lk, r)][row] = T{(double)acc_re[fm][fn][r], (double)acc_im[fm][fn][r]};
          else
            part[wk][wn * 16 + frag_col<TC>(lk, r)][row] = (double)acc_re[fm][fn][r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < (ENT + NTHR - 1) / NTHR; ++u) {
        const int e = threadIdx.x + u * NTHR;
        if (ENT % NTHR != 0 && e >= ENT) break;
        const int i = e % ROWS, c = e / ROWS;
        const int64_t nc = n0 + (c / 16) * FN * 16;
        const int64_t j = FB::index(nc, fn, c & 15, N);
        double cs = 0.0;
        if (m0 + i < M && FB::mine(nc, fn, c & 15, N)) {
          double vr = 0.0, vi = 0.0;
#pragma unroll
          for (int w = 0; w < WK; ++w) {
            const T v = part[w][c][i];
            vr += re_(v);
            vi += im_(v);
          }
          finish(m0 + i, j, vr, vi, cs, AHEAD ? &yc[fn][u] : nullptr);
        }
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
          for (int o = 1; o < ROWS; o *= 2) cs += __shfl_xor(cs, o, ROWS);
          if (i == 0 && FB::mine(nc, fn, c & 15, N)) csum[j - n0] = cs;
        }
      }
    }
    if constexpr (EPI == EPI_RESID) {
      __syncthreads();
      for (int e = threadIdx.x; e < TBN; e += NTHR)
        if (n0 + e < N) g.partial[(int64_t)tm * N + n0 + e] = csum[e];
    }
  } else {
    double colsum[FN][4];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) colsum[fn][r] = 0.0;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
      if (!FA::mine(mw, fm, l16, M)) continue;
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!FB::mine(nw, fn, frag_col<TC>(lk, r), N)) continue;
          double vi = 0.0;
          if constexpr (CPLX) vi = (double)acc_im[fm][fn][r];
          finish(FA::index(mw, fm, l16, M), FB::index(nw, fn, frag_col<TC>(lk, r), N),
                 (double)acc_re[fm][fn][r], vi, colsum[fn][r], nullptr);
        }
    }
    if constexpr (EPI == EPI_RESID) {
      __shared__ double red[WM][TBN];
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double v = colsum[fn][r];
          v += __shfl_xor(v, 1, 16);
          v += __shfl_xor(v, 2, 16);
          v += __shfl_xor(v, 4, 16);
          v += __shfl_xor(v, 8, 16);
          static_assert(EPI != EPI_RESID || !FB::PAIR, "columns of a residual are not paired");
          if (l16 == 0) red[wm][(wn * FN + fn) * 16 + frag_col<TC>(lk, r)] = v;
        }
      __syncthreads();
      for (int e = threadIdx.x; e < TBN; e += NTHR) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < WM; ++w) sum += red[w][e];
        if (n0 + e < N) g.partial[(int64_t)tm * N + n0 + e] = sum;
      }
    }
  }
}

template <typename TA, typename TC, bool CPLX, int OPA, int OPB, int EPI, bool G3, int FM, int FN,
          int WK = 8, int OCC = 1, int WM = 1, int WN = 1>
void launch(const GemmArgs& g, hipStream_t st) {
  constexpr int TBM = WM * FM * 16, TBN = WN * FN * 16;
  const int64_t tiles_m = (g.M + TBM - 1) / TBM;
  const int64_t tiles_n = (g.N + TBN - 1) / TBN;
  int64_t ntiles = tiles_m * tiles_n;
  if (EPI == EPI_SPLITK && g.tri) {
    CHASE_REQUIRE(g.M == g.N && TBM == TBN, "triangular split-K needs a square result");
    ntiles = tiles_m * (tiles_m + 1) / 2;
  }
  CHASE_REQUIRE(ntiles <= INT32_MAX - 8, "too many output tiles");
  const int grid_x = (int)((ntiles + 7) / 8 * 8);
  dim3 grid(grid_x, 1, EPI == EPI_SPLITK ? g.splits : 1);
  hipLaunchKernelGGL((gemm_kernel<TA, TC, CPLX, OPA, OPB, EPI, G3, FM, FN, WM, WN, WK, 2, OCC>),
                     grid, dim3(64 * WM * WN * WK), 0, st, g, (int)tiles_n, (int)ntiles);
  CHASE_HIP(hipGetLastError());
}

// Choice of the tile.  A workgroup's tile takes a compute unit a time
// proportional to its area divided by the rate `rate` the tile size reaches
// on a full chip (larger tiles load less per MFMA), and the busiest unit
// works through ceil(tiles / 256) of them: the tile with the least of that
// product is taken, the earlier one on a tie.
struct Tile {
  int tm, tn;
  double rate;
};
inline int64_t tiles_of(int64_t M, int64_t N, int tm, int tn) {
  return ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
}
inline double tile_cost(const Tile& t, int64_t M, int64_t N) {
  return (double)((tiles_of(M, N, t.tm, t.tn) + NCU - 1) / NCU) * t.tm * t.tn / t.rate;
}
template <int N>
int pick(const Tile (&t)[N], int64_t M, int64_t N_, double* least = nullptr) {
  int best = 0;
  double cost = 0.0;
  for (int i = 0; i < N; ++i) {
    const double c = tile_cost(t[i], M, N_);
    if (i == 0 || c < cost) {
      best = i;
      cost = c;
    }
  }
  if (least) *least = cost;
  return best;
}

// Complex, three-product form.  Rates: TFLOP/s (algorithmic) on the 20000 x
// 1300 filter step.  The smaller tiles earn their place where a dimension is
// ragged or the chip is not full: 1000 x 140 takes 22 us with 48 x 16 (189
// tiles), 28 with 32 x 32 (160) or 32 x 16 (288), 41 with 48 x 32 (105).  80 x 16
// against the best other tile: 3020 x 95 91 / 104 us, 2503 x 105 79 / 88, 1389 x
// 195 47 / 53, 3473 x 172 211 / 223, 1862 x 310 117 / 118.
// Splitting K over workgroups as well, the last one to arrive adding up the
// partial tiles, took 2 to 4 times as long as the best of these: the
// device-wide fences it needs write back the L2s.
template <int EPI>
void gauss_f64(const GemmArgs& g, hipStream_t st) {
  static constexpr Tile t[] = {{96, 32, 88}, {48, 32, 83}, {32, 32, 79}, {48, 16, 74},
                               {32, 16, 62}, {16, 16, 42}, {80, 16, 74}};
  switch (pick(t, g.M, g.N)) {
    case 0: return launch<double, double, true, OP_N, OP_N, EPI, true, 3, 2, 4, 1, 2>(g, st);
    case 1:
      // two workgroups of 4 waves a compute unit: one runs while the other
      // reduces and stores (82 -> 83); a single one needs 8 for two waves a
      // SIMD
      if (tiles_of(g.M, g.N, 48, 32) <= NCU)
        return launch<double, double, true, OP_N, OP_N, EPI, true, 3, 2>(g, st);
      return launch<double, double, true, OP_N, OP_N, EPI, true, 3, 2, 4, 2>(g, st);
    case 2: return launch<double, double, true, OP_N, OP_N, EPI, true, 2, 2>(g, st);
    case 3: return launch<double, double, true, OP_N, OP_N, EPI, true, 3, 1>(g, st);
    case 4: return launch<double, double, true, OP_N, OP_N, EPI, true, 2, 1>(g, st);
    case 6: return launch<double, double, true, OP_N, OP_N, EPI, true, 5, 1>(g, st);
    default: return launch<double, double, true, OP_N, OP_N, EPI, true, 1, 1>(g, st);
  }
}

// Real rank-k updates on 64 x 32 tiles of two waves a K half (rank_tile): where
// the 32 x 32 tiles would fill the chip and up to this rank.  Against the tiles
// of the table below, us: order 2000 rank 400 60 / 70, 700 98 / 102; 3500: 173 /
// 187, 291 / 283; 20000: 5355 / 5895, 8769 / 8883, but 7685 / 7199 at 512.
constexpr int64_t kRankK = 448;
inline bool rank_tile(const GemmArgs& g) {
  return std::max(g.K, g.K2) <= kRankK && tiles_of(g.M, g.N, 32, 32) >= 4 * NCU;
}

// Waves per workgroup of the four-product and residual forms' 32 x 32 tiles:
// 8 while the tiles do not fill the chip; with 1024 tiles or more (four 4-wave
// workgroups a compute unit), fewer waves split K, so that more workgroups
// overlap one's reduction and stores with another's products.  8000 x 260 x
// 260: 87 us with 8, 78 with 4; rank-96 update of order 3000: 201 / 138 / 126
// us with 8 / 4 / 2, rank-960: 1084 / 982 / 1005.  About the line, complex rank-k
// updates with 4 / 2 waves, us: order 1100, rank 100 27 / 27, 192 37 / 42, 260 47 /
// 54; 5000: 192 609 / 589, 260 790 / 780; 20000: 192 9470 / 9020, 500 22680 / 22500:
// beyond it two waves cost a small order up to 15% and gain a large one 2%.
inline int waves_of(const GemmArgs& g) {
  if (tiles_of(g.M, g.N, 32, 32) < 4 * NCU) return 8;
  return g.K <= 192 ? 2 : 4;
}

// Two rank-k updates of one matrix in one pass (K2 > 0): on the two-wave
// tile, a wave each, where that tile fills the chip; the matrix is read and
// written once instead of twice (two rank-96 updates of order 3000, complex,
// between filter steps: 306 -> 253 us).  The real update takes it only where
// its single ones run on the same tile.
inline bool rank_pair(bool cplx, const GemmArgs& g) {
  if (g.M < 2 || g.N < 2 || tiles_of(g.M, g.N, 32, 32) < 4 * NCU) return false;
  return cplx || rank_tile(g);
}

// Complex, four-product form.  Rates: 20000 x 1300 x 1300.
template <int OPA, int OPB, int EPI>
void four_f64(const GemmArgs& g, hipStream_t st) {
  static constexpr Tile t[] = {{32, 32, 66}, {16, 16, 45}, {64, 32, 71}};
  constexpr int OCC = OPB == OP_C ? 3 : 4;
  const int p = pick(t, g.M, g.N);
  if (p == 1) return launch<double, double, true, OPA, OPB, EPI, false, 1, 1>(g, st);
  // the larger tile for long blocks times a factor only: the rank-k updates
  // (OPB = C) are short and bound by C, and the shifted products with H (SHIFT),
  // long in K, gain nothing (eigenvector adjoint 12000 x 300: 178 ms with 32 x
  // 32, 185 with 64 x 32; 8000 x 1500: 478 and 472)
  if constexpr (OPB == OP_N && EPI != EPI_SHIFT) {
    if (p == 2) return launch<double, double, true, OPA, OPB, EPI, false, 4, 2, 4, 2>(g, st);
  }
  switch (waves_of(g)) {
    case 2: return launch<double, double, true, OPA, OPB, EPI, false, 2, 2, 2, OCC>(g, st);
    case 4: return launch<double, double, true, OPA, OPB, EPI, false, 2, 2, 4, OCC>(g, st);
    default: return launch<double, double, true, OPA, OPB, EPI, false, 2, 2>(g, st);
  }
}

// Real.  Rates: TFLOP/s on a 10000 x 1024 filter step; 2000 x 100 takes 21 us
// with 64 x 16 (224 tiles), 23 with 32 x 32 (252), 37 with 64 x 32 (128).
template <int OPA, int OPB, int EPI>
void real_f64(const GemmArgs& g, hipStream_t st) {
  // pairs of rows (or columns) are loaded together: at least two of them
  if (g.M < 2 || g.N < 2)
    return launch<double, double, false, OPA, OPB, EPI, false, 1, 1>(g, st);
  // rank-k updates (order 2000, rank 100: 25 us; 28 on 32 x 32 tiles, 33 with
  // 64 x 32 tiles and four waves that split K)
  if constexpr (OPB == OP_C) {
    if (rank_tile(g))
      return launch<double, double, false, OPA, OPB, EPI, false, 2, 2, 2, 4, 2>(g, st);
  } else {
    // a long block times a small factor: short K, see waves_of
    if (g.K <= 192 && waves_of(g) == 2)
      return launch<double, double, false, OPA, OPB, EPI, false, 2, 2, 2, 4>(g, st);
  }
  static constexpr Tile t[] = {{128, 64, 70}, {64, 64, 67}, {64, 32, 62}, {64, 16, 55},
                               {32, 32, 48},  {32, 16, 41}, {16, 16, 24}, {96, 32, 64}};
  switch (pick(t, g.M, g.N)) {
    case 0: return launch<double, double, false, OPA, OPB, EPI, false, 4, 4, 2, 2, 2>(g, st);
    case 1:
      // a single workgroup a compute unit needs 8 waves for two a SIMD (5003
      // x 173: 161 us with 4, 157 with 8)
      if (tiles_of(g.M, g.N, 64, 64) <= NCU)
        return launch<double, double, false, OPA, OPB, EPI, false, 4, 4>(g, st);
      return launch<double, double, false, OPA, OPB, EPI, false, 4, 4, 4, 2>(g, st);
    case 2: return launch<double, double, false, OPA, OPB, EPI, false, 4, 2, 4, 3>(g, st);
    case 3: return launch<double, double, false, OPA, OPB, EPI, false, 4, 1>(g, st);
    case 4: return launch<double, double, false, OPA, OPB, EPI, false, 2, 2>(g, st);
    case 5: return launch<double, double, false, OPA, OPB, EPI, false, 2, 1>(g, st);
    case 7: return launch<double, double, false, OPA, OPB, EPI, false, 6, 2>(g, st);
    default: return launch<double, double, false, OPA, OPB, EPI, false, 1, 1>(g, st);
  }
}

// ------------------------------------------------------------------ staged FP32
// FP32 filter step through LDS: 128 x 64 tiles, K chunks of 16 in two stages, 512
// threads = 8 waves of 32 x 32 (4 x 2); the next chunk's loads are in flight
// during a chunk's MFMAs, operands are rounded to FP32 on the way into LDS
// (k-major, one element of padding a row against bank conflicts).  A thread's
// loads run along the columns of A and B whatever their alignment, and each
// element is read once per tile: where the direct kernel's fragment loads are
// the bound (wide blocks, columns that do not begin on a cache line, H in
// FP64), this one is faster (see cheb_f32).
constexpr int STM = 128, STN = 64, SBK = 16, SNT = 512, SPAD = 1;

template <typename TA, bool CPLX>
__global__ __launch_bounds__(SNT) void staged_f32_kernel(GemmArgs g, int tiles_n, int ntiles) {
  using TE = typename El<double, CPLX>::type;  // element of B and C
  using TAe = typename El<TA, CPLX>::type;
  using V = typename El<float, CPLX>::type;
  constexpr int LA = STM * SBK / SNT, LB = STN * SBK / SNT;  // elements a thread loads
  __shared__ V As[2][SBK][STM + SPAD];
  __shared__ V Bs[2][SBK][STN + SPAD];
  const int per_xcd = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= ntiles) return;
  const int tm = t / tiles_n, tn = t - tm * tiles_n;
  const int64_t m0 = (int64_t)tm * STM, n0 = (int64_t)tn * STN, M = g.M, N = g.N, K = g.K;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lk = lane >> 4;
  const TAe* __restrict__ A = static_cast<const TAe*>(g.A);
  const TE* __restrict__ B = static_cast<const TE*>(g.B);

  TAe ra[LA];
  TE rb[LB];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int e = 0; e < LA; ++e) {
      const int idx = tid + e * SNT;
      const int64_t i = m0 + idx % STM, k = k0 + idx / STM;
      ra[e] = i < M && k < K ? A[i + k * g.lda] : TAe(0);
    }
#pragma unroll
    for (int e = 0; e < LB; ++e) {
      const int idx = tid + e * SNT;
      const int64_t k = k0 + idx % SBK, j = n0 + idx / SBK;
      rb[e] = j < N && k < K ? B[k + j * g.ldb] : TE(0);
    }
  };
  auto rounded = [](auto x) {
    if constexpr (CPLX)
      return V{(float)x.x, (float)x.y};
    else
      return (float)x;
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < LA; ++e) {
      const int idx = tid + e * SNT;
      As[buf][idx / STM][idx % STM] = rounded(ra[e]);
    }
#pragma unroll
    for (int e = 0; e < LB; ++e) {
      const int idx = tid + e * SNT;
      Bs[buf][idx % SBK][idx / SBK] = rounded(rb[e]);
    }
  };

  // complex: re*re, im*im and (re + im)(re + im)
  f4 p1[2][2], p2[CPLX ? 2 : 1][2], p3[CPLX ? 2 : 1][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      p1[a][b] = f4{0, 0, 0, 0};
      if constexpr (CPLX) p2[a][b] = p3[a][b] = f4{0, 0, 0, 0};
    }
  const int64_t nchunks = (K + SBK - 1) / SBK;
  load(0);
  store(0);
  __syncthreads();
  for (int64_t c = 0; c < nchunks; ++c) {
    const int buf = (int)(c & 1);
    const bool more = c + 1 < nchunks;
    if (more) load((c + 1) * SBK);
#pragma unroll
    for (int ks = 0; ks < SBK / 4; ++ks) {
      const int kk = ks * 4 + lk;
      V a[2], b[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        a[f] = As[buf][kk][wm * 32 + f * 16 + l16];
        b[f] = Bs[buf][kk][wn * 32 + f * 16 + l16];
      }
#pragma unroll
      for (int fn = 0; fn < 2; ++fn)
#pragma unroll
        for (int fm = 0; fm < 2; ++fm) {
          if constexpr (CPLX) {
            p1[fm][fn] = MF<float>::fma(b[fn].x, a[fm].x, p1[fm][fn]);
            p2[fm][fn] = MF<float>::fma(b[fn].y, a[fm].y, p2[fm][fn]);
            p3[fm][fn] = MF<float>::fma(b[fn].x + b[fn].y, a[fm].x + a[fm].y, p3[fm][fn]);
          } else {
            p1[fm][fn] = MF<float>::fma(b[fn], a[fm], p1[fm][fn]);
          }
        }
    }
    if (more) store(buf ^ 1);
    __syncthreads();
  }

  TE* __restrict__ C = static_cast<TE*>(g.C);
#pragma unroll
  for (int fm = 0; fm < 2; ++fm) {
    const int64_t i = m0 + wm * 32 + fm * 16 + l16;
    if (i >= M) continue;
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = n0 + wn * 32 + fn * 16 + frag_col<float>(lk, r);
        if (j >= N) continue;
        double vr = (double)p1[fm][fn][r], vi = 0.0;
        if constexpr (CPLX) {
          const float q1 = p1[fm][fn][r], q2 = p2[fm][fn][r];
          vr = (double)(q1 - q2);
          vi = (double)(p3[fm][fn][r] - q1 - q2);
        }
        const TE x = B[i + j * g.ldb];
        vr = g.alpha * (vr - g.gamma * re_(x));
        vi = g.alpha * (vi - g.gamma * im_(x));
        if (g.beta != 0.0) {
          const TE y = C[i + j * g.ldc];
          vr += g.beta * re_(y);
          vi += g.beta * im_(y);
        }
        if (g.colcoef) {
          const double cj = g.colcoef[j];
          const TE f = static_cast<const TE*>(g.F)[i + j * g.ldf];
          vr += cj * re_(f);
          vi += cj * im_(f);
        }
        if constexpr (CPLX)
          C[i + j * g.ldc] = TE{vr, vi};
        else
          C[i + j * g.ldc] = vr;
      }
  }
}

template <typename TA, bool CPLX>
void launch_staged_f32(const GemmArgs& g, hipStream_t st) {
  const int64_t tiles_n = (g.N + STN - 1) / STN, ntiles = (g.M + STM - 1) / STM * tiles_n;
  CHASE_REQUIRE(ntiles <= INT32_MAX - 8, "too many output tiles");
  hipLaunchKernelGGL((staged_f32_kernel<TA, CPLX>), dim3((unsigned)((ntiles + 7) / 8 * 8)),
                     dim3(SNT), 0, st, g, (int)tiles_n, (int)ntiles);
  CHASE_HIP(hipGetLastError());
}

// Whether the direct kernel's speed suffers from columns that do not begin at
// multiples of 32 bytes, 64 for H in FP64 (odd orders): 20001 rows against 20000,
// 1300 columns, 35.0 ms instead of 27.9 complex and 16.1 instead of 10.9 real, the
// staged kernel 28.1 (28.0) and 11.8 (11.5).  Smaller matrices and blocks lose less
// than the direct tiles' finer division gains; direct / staged, passes of degrees
// 2 to 10, ms: complex 9001 x 900 33.5 / 35.5, 11001 x 400 22.3 / 25.2, 10007 x 1001
// 43.9 / 41.2, 20001 x 400 92.2 / 85.2; real 11001 x 400 10.5 / 11.0, 20001 x 300
// 30.4 / 29.5; H in FP64, complex 20001 x 300 89.0 / 73.5, real 9001 x 900 18.9 / 17.2.
template <typename TA, bool CPLX>
bool f32_unaligned(const GemmArgs& g) {
  constexpr int64_t W = CPLX ? 2 : 1;
  constexpr int64_t line = sizeof(TA) == 8 ? 64 : 32;
  if (g.lda * W * (int64_t)sizeof(TA) % line == 0 && g.ldb * W * 8 % line == 0) return false;
  if (sizeof(TA) == 8) return g.M >= (CPLX ? 9600 : 8000);
  return CPLX ? g.M >= 9600 && g.M * g.N >= 7000000 : g.M * g.N >= 5500000;
}
// The staged kernel with `rate`, where it has two tiles for every compute unit
// (with H in FP64 for half of them) and undercuts the direct tiles' cost.  20001 x
// 150, 471 tiles, pass of degrees 2 to 10, direct / staged: real 17.2 / 18.7 ms,
// with H in FP64 21.2 / 19.8.
template <typename TA>
bool staged_f32(const GemmArgs& g, double rate, double direct) {
  const Tile t{STM, STN, rate};
  return 2 * tiles_of(g.M, g.N, STM, STN) >= (sizeof(TA) == 8 ? 3 : 4) * NCU &&
         tile_cost(t, g.M, g.N) < direct;
}

// FP32 products of the filter step (A stored as TA, B in FP64), complex.
// Rates: TFLOP/s (algorithmic) on the 20000 x 1300 step; 8000 x 260 takes 1.03
// ms with 96 x 48 tiles, 1.08 with 64 x 32, 1.70 with 128 x 64.  H in FP64 (no
// room for its FP32 copy) doubles the bytes of its fragments: the staged kernel
// is the faster one there for wide blocks (20000 x 1300 29.2 ms, 31.1 with 96 x
// 48; 9000 x 700 4.20 and 3.63).
template <typename TA>
void cheb_f32_cplx(const GemmArgs& g, hipStream_t st) {
  static constexpr Tile t[] = {{128, 64, 150}, {64, 32, 146}, {32, 32, 96}, {32, 16, 81},
                               {16, 16, 47}, {96, 48, 146}};
  static constexpr Tile t64[] = {{128, 64, 136}, {64, 32, 134}, {32, 32, 96}, {32, 16, 81},
                                 {16, 16, 47}, {96, 48, 139}};
  static constexpr Tile tu[] = {{128, 64, 120}, {64, 32, 108}, {32, 32, 65}, {32, 16, 55},
                                {16, 16, 35}, {96, 48, 116}};
  const bool unaligned = f32_unaligned<TA, true>(g);
  double c;
  const int p = unaligned ? pick(tu, g.M, g.N, &c)
                : sizeof(TA) == 8 ? pick(t64, g.M, g.N, &c) : pick(t, g.M, g.N, &c);
  if ((unaligned || sizeof(TA) == 8) && staged_f32<TA>(g, 149, c))
    return launch_staged_f32<TA, true>(g, st);
  switch (p) {
    case 0: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 4, 2, 2, 1, 2, 2>(g, st);
    case 1: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 4, 2, 4, 2>(g, st);
    case 2: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 2, 2>(g, st);
    case 3: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 2, 1>(g, st);
    case 5: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 3, 3, 4, 1, 2>(g, st);
    default: return launch<TA, float, true, OP_N, OP_N, EPI_CHEB, true, 1, 1>(g, st);
  }
}

// Real: tables of their own (96 x 48 has an odd number of row fragments, and the
// rates are not in proportion).  Rates: TFLOP/s on steps of 4000 x 1000 to 20000
// x 1300.  15000 x 2000 takes 9.1 ms with 128 x 128, 10.6 with 128 x 64, 10.8
// with 64 x 32; 9000 x 1500 2.74, 2.88, 3.11.  H in FP64: 6001 x 1500 1.51 ms staged,
// 1.67 with 128 x 128; 9000 x 700 1.83 and 1.35.
template <typename TA>
void cheb_f32_real(const GemmArgs& g, hipStream_t st) {
  // pairs of rows are loaded together: at least two of them
  if (g.M < 2) return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 1, 1>(g, st);
  static constexpr Tile t[] = {{128, 128, 97}, {128, 64, 88}, {64, 32, 80},
                               {32, 32, 46},   {32, 16, 44},  {16, 16, 23}};
  static constexpr Tile t64[] = {{128, 128, 92}, {128, 64, 80}, {64, 32, 68},
                                 {32, 32, 44},   {32, 16, 42},  {16, 16, 22}};
  static constexpr Tile tu[] = {{128, 128, 68}, {128, 64, 65},
                                {64, 32, sizeof(TA) == 8 ? 60 : 65},
                                {32, 32, 38}, {32, 16, 36}, {16, 16, 20}};
  const bool unaligned = f32_unaligned<TA, false>(g);
  double c;
  const int p = unaligned ? pick(tu, g.M, g.N, &c)
                : sizeof(TA) == 8 ? pick(t64, g.M, g.N, &c) : pick(t, g.M, g.N, &c);
  if ((unaligned || sizeof(TA) == 8) && staged_f32<TA>(g, sizeof(TA) == 8 ? 83 : 90, c))
    return launch_staged_f32<TA, false>(g, st);
  switch (p) {
    case 0: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 4, 4, 2, 1, 2, 2>(g, st);
    case 1: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 4, 2, 2, 1, 2, 2>(g, st);
    case 2: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 4, 2, 4, 2>(g, st);
    case 3: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 2, 2>(g, st);
    case 4: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 2, 1>(g, st);
    default: return launch<TA, float, false, OP_N, OP_N, EPI_CHEB, false, 1, 1>(g, st);
  }
}

constexpr int kResidRows = 32;  // row tile of EPI_RESID

template <bool CPLX>
void dispatch(Prec prec, Op opa, Op opb, Epi epi, const GemmArgs& g, hipStream_t st) {
  if (prec == PREC_F32) {
    CHASE_REQUIRE(opa == OP_N && opb == OP_N && epi == EPI_CHEB,
                  "FP32 products exist only for the filter step");
    if constexpr (CPLX)
      return g.a_f32 ? cheb_f32_cplx<float>(g, st) : cheb_f32_cplx<double>(g, st);
    else
      return g.a_f32 ? cheb_f32_real<float>(g, st) : cheb_f32_real<double>(g, st);
  }
  if (opa == OP_N && opb == OP_N) {
    switch (epi) {
      case EPI_STORE:
        // long products (H times a block) use the three-product form as the
        // filter does; the short ones of QR and Rayleigh-Ritz keep four
        if constexpr (CPLX) {
          if (g.K >= 4096) return gauss_f64<EPI_STORE>(g, st);
          return four_f64<OP_N, OP_N, EPI_STORE>(g, st);
        } else {
          return real_f64<OP_N, OP_N, EPI_STORE>(g, st);
        }
      case EPI_CHEB:
        if constexpr (CPLX)
          return gauss_f64<EPI_CHEB>(g, st);
        else
          return real_f64<OP_N, OP_N, EPI_CHEB>(g, st);
      case EPI_RESID:
        // 32-row tiles at any size: one partial norm per column and tile.  A
        // single row (the lanes' row pairs need two) runs on 16-row tiles.
        if (!CPLX && g.M < 2)
          return launch<double, double, CPLX, OP_N, OP_N, EPI_RESID, false, 1, 1>(g, st);
        if (waves_of(g) == 8)
          return launch<double, double, CPLX, OP_N, OP_N, EPI_RESID, false, 2, 2>(g, st);
        return launch<double, double, CPLX, OP_N, OP_N, EPI_RESID, false, 2, 2, 4, 4>(g, st);
      case EPI_SHIFT:
        if constexpr (CPLX)
          return four_f64<OP_N, OP_N, EPI_SHIFT>(g, st);
        else
          return real_f64<OP_N, OP_N, EPI_SHIFT>(g, st);
      default: break;
    }
  } else if (opa == OP_C && opb == OP_N) {
    if (epi == EPI_SPLITK) {
      if constexpr (CPLX) {
        return launch<double, double, CPLX, OP_C, OP_N, EPI_SPLITK, false, 2, 2>(g, st);
      } else {
        if (splitk_tile(CPLX, g.M, g.K) == 64)
          return launch<double, double, CPLX, OP_C, OP_N, EPI_SPLITK, false, 4, 4, 4, 2>(g, st);
        return launch<double, double, CPLX, OP_C, OP_N, EPI_SPLITK, false, 2, 2>(g, st);
      }
    }
  } else if (opa == OP_N && opb == OP_C && epi == EPI_STORE) {
    if constexpr (CPLX)
      return four_f64<OP_N, OP_C, EPI_STORE>(g, st);
    else
      return real_f64<OP_N, OP_C, EPI_STORE>(g, st);
  }
  throw Error(CHASE_ERR_ARG, "unsupported GEMM form");
}

}  // namespace

int gemm_row_tiles(int64_t M) { return (int)((M + kResidRows - 1) / kResidRows); }

// Square tile of the split-K products: 32 for complex data; real data reaches
// 60 TFLOP/s with 64 and 36 with 32 (20000 x 1300), as long as the tiles and
// the K slices of 256 give every compute unit a workgroup.
int splitk_tile(bool cplx, int64_t M, int64_t K) {
  const int64_t tm = (M + 63) / 64;
  return cplx || M <= 32 || tm * (tm + 1) / 2 * (K / 256) < NCU ? 32 : 64;
}

// Slices: about 1024 workgroups of a few waves, at least four slices where
// the tiles alone are no more than that (the last, partly filled round costs
// less: 20000 x 1300 complex 2.56 ms with one slice, 2.14 with four), but not more than 4096 in all; each slice at least 256 long.  tri:
// the tiles on and above the diagonal only.
void splitk_plan(bool cplx, int64_t M, int64_t N, int64_t K, int* splits, int64_t* kslice,
                 bool tri) {
  const int64_t T = splitk_tile(cplx, M, K);
  const int64_t tm = (M + T - 1) / T;
  const int64_t tiles = tri ? tm * (tm + 1) / 2 : tm * ((N + T - 1) / T);
  int64_t s = std::max((4 * NCU + tiles - 1) / tiles,
                       std::min<int64_t>(4, (16 * NCU + tiles - 1) / tiles));
  const int64_t smax = (K + 255) / 256;
  if (s > smax) s = smax;
  if (s < 1) s = 1;
  int64_t ks = (K + s - 1) / s;
  ks = (ks + 15) / 16 * 16;
  s = (K + ks - 1) / ks;
  if (s < 1) s = 1;
  *splits = (int)s;
  *kslice = ks;
}

void gemm(bool cplx, Prec prec, Op opa, Op opb, Epi epi, const GemmArgs& g, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0) return;
  if (is_split_bf16(prec)) {
    CHASE_REQUIRE(opa == OP_N && opb == OP_N && epi == EPI_CHEB,
                  "split-BF16 products exist only for the filter step");
    return gemm_bf16x3(cplx, g, st, prec == PREC_BF16X2 ? 2 : 3);
  }
  if (g.K2 > 0) {
    CHASE_REQUIRE(prec == PREC_F64 && opa == OP_N && opb == OP_C && epi == EPI_STORE,
                  "two products in one pass: rank-k updates only");
    if (rank_pair(cplx, g)) {
      if (cplx)
        launch<double, double, true, OP_N, OP_C, EPI_STORE, false, 2, 2, 2, 3>(g, st);
      else
        launch<double, double, false, OP_N, OP_C, EPI_STORE, false, 2, 2, 2, 4, 2>(g, st);
      return;
    }
    GemmArgs g1 = g, g2 = g;
    g1.K2 = g2.K2 = 0;
    g2.A = g.A2;
    g2.lda = g.lda2;
    g2.B = g.B2;
    g2.ldb = g.ldb2;
    g2.K = g.K2;
    g2.alpha = g.alpha * g.ratio2;
    g2.beta = 1.0;
    gemm(cplx, prec, opa, opb, epi, g1, st);
    return gemm(cplx, prec, opa, opb, epi, g2, st);
  }
  if (cplx)
    dispatch<true>(prec, opa, opb, epi, g, st);
  else
    dispatch<false>(prec, opa, opb, epi, g, st);
}

}  // namespace chase
