// Dense Hermitian eigensolver of the Rayleigh-Ritz step (Algorithm 1;
// Section 2.3: the projected matrix G = Q^H H Q is diagonalised), on the GPU.
//
// Block-cyclic two-sided Jacobi (Golub & Van Loan, symmetric Schur rotations
// with a parallel round-robin ordering, block form).  The k x k matrix is cut
// into blocks of JB indices.  A sweep is the round-robin tournament over the
// blocks: in each round every pair of blocks (p, q) gets one cyclic Jacobi
// sweep over its 2 JB indices, run by one workgroup in LDS and accumulated
// into a 2JB x 2JB unitary U_pq; the next round's launch applies all pairs' U
// to the whole matrix (G <- J^H G J, J the block-diagonal product of the U_pq)
// and to the eigenvector block (V <- V J) beside its own pairs, which form
// their subproblems themselves.  The convergence is quadratic; in the
// subspace iteration the projected matrix is close to diagonal once the
// Ritz vectors settle, and then a few sweeps suffice.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <utility>

namespace chase {
namespace {

constexpr int JB = 16;       // indices per block
constexpr int JM = 2 * JB;   // order of a pair's subproblem
constexpr int JLD = JM + 1;  // LDS leading dimension (padded against bank conflicts)
constexpr int JT = 256;      // threads per workgroup
constexpr int JPT = 2 * JT;  // threads per workgroup of the pair solves
constexpr int NPART = 256;   // workgroups of the norm reduction

struct cd {
  double x, y;
};
__device__ __forceinline__ cd operator+(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cd operator-(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cd operator*(cd a, cd b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
__device__ __forceinline__ cd operator*(cd a, double s) { return {a.x * s, a.y * s}; }
__device__ __forceinline__ double conj_(double a) { return a; }
__device__ __forceinline__ cd conj_(cd a) { return {a.x, -a.y}; }
__device__ __forceinline__ double abs2(double a) { return a * a; }
__device__ __forceinline__ double abs2(cd a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ double real_(double a) { return a; }
__device__ __forceinline__ double real_(cd a) { return a.x; }
template <class T>
__device__ __forceinline__ T from_real(double a);
template <>
__device__ __forceinline__ double from_real<double>(double a) { return a; }
template <>
__device__ __forceinline__ cd from_real<cd>(double a) { return {a, 0.0}; }
// Round-robin tournament over m players (m even), rounds r = 0 .. m-2:
// player 0 stays, the others rotate; pair t of round r is
// (rr_player(m, r, t), rr_player(m, r, m - 1 - t)).  Over the m - 1 rounds
// every two players meet exactly once.
__host__ __device__ inline int rr_player(int m, int r, int j) {
  return j == 0 ? 0 : (j - 1 + r) % (m - 1) + 1;
}

// Pair of round r that player x (of m) is in, and whether as its first (0) or
// second (1) player: the inverse of rr_player.
__device__ inline void rr_place(int m, int r, int x, int& pair, int& half) {
  const int j = x == 0 ? 0 : (x - 1 + (m - 1) - r) % (m - 1) + 1;
  half = j >= m / 2;
  pair = half ? m - 1 - j : j;
}

// Value of the next and of the previous lane of the 16-lane DPP row (the row's
// last and first lane: 0).
__device__ __forceinline__ double from_lane_above(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x101, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x101, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_lane_below(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x111, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x111, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ cd from_lane_above(cd v) {
  return {from_lane_above(v.x), from_lane_above(v.y)};
}
__device__ __forceinline__ cd from_lane_below(cd v) {
  return {from_lane_below(v.x), from_lane_below(v.y)};
}
__device__ __forceinline__ double pick(bool c, double a, double b) { return c ? a : b; }
__device__ __forceinline__ cd pick(bool c, cd a, cd b) {
  return {c ? a.x : b.x, c ? a.y : b.y};
}

// Player of an inner round (m = JM, 0 <= r < JM - 1) without a division.
__device__ __forceinline__ int inner_player(int r, int j) {
  const int p = j - 1 + r;
  return j == 0 ? 0 : p >= JM - 1 ? p - (JM - 2) : p + 1;
}

// Rotation that zeroes the (a, b) entry of the 2 x 2 Hermitian
// [[app, apq], [conj(apq), aqq]]: with apq = g ph (g = |apq|, |ph| = 1),
// u = [[cs, sn], [-sn conj(ph), cs conj(ph)]] = diag(1, conj(ph)) R, R the
// real rotation [[cs, sn], [-sn, cs]] by the smaller of the two angles, and
// u^H A u is diagonal: with d = aqq - app and h = sqrt(d^2 + 4 g^2), the double
// angle has cosine |d| / h and sine 2 g / h, so cs^2 = (1 + |d| / h) / 2 and
// sn = sign(d) g / (h cs): two reciprocal square roots on the dependent path,
// no division.
// Entries with g <= thr are left alone (identity).
template <class T>
__device__ __forceinline__ int jac_rotation(double app, double aqq, T apq, double thr, double& cs,
                                            double& sn, T& ph) {
  const double g2 = abs2(apq);
  if (!(g2 > thr * thr)) {
    cs = 1.0;
    sn = 0.0;
    ph = from_real<T>(1.0);
    return 0;
  }
  const double d = aqq - app;
  const double rh = rsqrt(fma(d, d, 4.0 * g2));
  const double rg = rsqrt(g2);
  const double c2 = fma(0.5 * fabs(d), rh, 0.5);  // cs^2, in [1/2, 1]
  const double rc = rsqrt(c2);
  cs = c2 * rc;
  sn = copysign(g2 * rg * rh * rc, d);
  ph = apq * rg;
  return 1;
}

typedef double d4v __attribute__((ext_vector_type(4)));

// Y = A B for JM x JM tiles in LDS on the FP64 matrix cores (16x16x4 MFMA),
// A(i, l) at As[l * JLD + i] and B(l, c) at Bs[l * JLD + c].  Wave w of the
// four computes the quadrant of rows 16 (w & 1) and columns 16 (w >> 1).
// The operands go in swapped (B first), so the instruction produces the
// quadrant transposed: lane L holds Y(16 (w & 1) + L % 16, 16 (w >> 1) +
// L / 16 + 4 r) in out[r] (rows run along the lanes, as stores want them).
__device__ __forceinline__ void tile_mma(const double* As, const double* Bs, double (&out)[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i0 = 16 * (w & 1), c0 = 16 * (w >> 1), l16 = lane & 15, lk = lane >> 4;
  d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k0 = 0; k0 < JM; k0 += 4) {
    const double a = As[(k0 + lk) * JLD + i0 + l16];
    const double b = Bs[(k0 + lk) * JLD + c0 + l16];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b, a, acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) out[r] = acc[r];
}
__device__ __forceinline__ void tile_mma(const cd* As, const cd* Bs, cd (&out)[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i0 = 16 * (w & 1), c0 = 16 * (w >> 1), l16 = lane & 15, lk = lane >> 4;
  d4v re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k0 = 0; k0 < JM; k0 += 4) {
    const cd a = As[(k0 + lk) * JLD + i0 + l16];
    const cd b = Bs[(k0 + lk) * JLD + c0 + l16];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(b.x, a.x, re, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-b.y, a.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(b.y, a.x, im, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(b.x, a.y, im, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) out[r] = cd{re[r], im[r]};
}

// Position of out[r] of tile_mma in this thread: row, column.
__device__ __forceinline__ int mma_row() { return 16 * ((threadIdx.x >> 6) & 1) + (threadIdx.x & 15); }
__device__ __forceinline__ int mma_col(int r) {
  return 16 * (threadIdx.x >> 7) + ((threadIdx.x & 63) >> 4) + 4 * r;
}

// One 16 x 16 product over JM = 32 terms on the FP64 matrix cores: C(r, c) =
// sum_l a(l, r) b(l, c), from the lane's a(4 s + L / 16, L % 16) and b(4 s + L
// / 16, L % 16), s = 0 .. 7; lane L gets C(L % 16, L / 16 + 4 q) in out[q]
// (operands swapped as in tile_mma).
__device__ __forceinline__ void quad_mma(const double (&a)[JM / 4], const double (&b)[JM / 4],
                                         double (&out)[4]) {
  d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < JM / 4; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s], a[s], acc, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) out[q] = acc[q];
}
__device__ __forceinline__ void quad_mma(const cd (&a)[JM / 4], const cd (&b)[JM / 4],
                                         cd (&out)[4]) {
  d4v re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < JM / 4; ++s) {
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s].x, a[s].x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s].y, a[s].x, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-b[s].y, a[s].y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s].x, a[s].y, im, 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) out[q] = cd{re[q], im[q]};
}

constexpr int THLD = JB + 1;  // row length of the half tiles in pair_load

// The subproblem of blocks (bp, bq) after the rotations of round `prev`, from
// the matrix before them: bp was in pair x of that round (indices X), bq in
// pair y (indices Y), x != y as two blocks meet once a sweep, so
//   S = [ Ux' G(X,X) Ux, Ux' G(X,Y) Uy; ., Uy' G(Y,Y) Uy ]
// with the JB columns of Ux and Uy that belong to bp and bq.  Six waves form
// the three right products (32 x 16, one 16-row half each) straight from
// global memory, three the left ones.  Ts: 3 * JM * THLD elements.
template <class T>
__device__ void pair_load(const T* __restrict__ G, int64_t ldg, int k, int nb, int prev, int bp,
                          int bq, const T* __restrict__ uprev, T* S, T* Ts) {
  int x, hx, y, hy;
  rr_place(nb, prev, bp, x, hx);
  rr_place(nb, prev, bq, y, hy);
  const int x0 = rr_player(nb, prev, x), x1 = rr_player(nb, prev, nb - 1 - x);
  const int y0 = rr_player(nb, prev, y), y1 = rr_player(nb, prev, nb - 1 - y);
  const T* Ux = uprev + (int64_t)x * JM * JM + hx * JB * JM;  // its JB columns
  const T* Uy = uprev + (int64_t)y * JM * JM + hy * JB * JM;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  if (w < 6) {
    const int s = w >> 1;  // product: (X,X), (X,Y), (Y,Y)
    const int rh = w & 1;  // 16-row half
    const int gr = (s < 2 ? (rh ? x1 : x0) : (rh ? y1 : y0)) * JB + l16;
    const int c0 = s == 0 ? x0 : y0, c1 = s == 0 ? x1 : y1;
    const T* Ub = s == 0 ? Ux : Uy;
    T a[JM / 4], b[JM / 4], out[4];
#pragma unroll
    for (int st = 0; st < JM / 4; ++st) {
      const int l = 4 * st + lk;
      const int gc = (st < JM / 8 ? c0 : c1) * JB + (l & (JB - 1));
      a[st] = gr < k && gc < k ? G[gr + (int64_t)gc * ldg] : from_real<T>(0.0);
      b[st] = Ub[l + l16 * JM];
    }
    quad_mma(a, b, out);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      Ts[(s * JM + rh * JB + l16) * THLD + lk + 4 * q] = out[q];
  }
  __syncthreads();
  if (w < 3) {
    const T* Ua = w < 2 ? Ux : Uy;
    T a[JM / 4], b[JM / 4], out[4];
#pragma unroll
    for (int st = 0; st < JM / 4; ++st) {
      const int l = 4 * st + lk;
      a[st] = conj_(Ua[l + l16 * JM]);
      b[st] = Ts[(w * JM + l) * THLD + l16];
    }
    quad_mma(a, b, out);
    const int r0 = w < 2 ? 0 : JB, c0 = w < 1 ? 0 : JB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + l16, c = c0 + lk + 4 * q;
      S[c * JLD + r] = out[q];
      if (w == 1) S[r * JLD + c] = conj_(out[q]);
    }
  }
  __syncthreads();
  // the diagonal blocks Hermitian to the last bit, as the stored tiles are
  for (int e = threadIdx.x; e < 2 * JB * JB; e += JPT) {
    const int d = e / (JB * JB) * JB, r = d + e % JB, c = d + e % (JB * JB) / JB;
    if (r < c) {
      const T v = (S[c * JLD + r] + conj_(S[r * JLD + c])) * 0.5;
      S[c * JLD + r] = v;
      S[r * JLD + c] = conj_(v);
    } else if (r == c) {
      S[c * JLD + r] = from_real<T>(real_(S[c * JLD + r]));
    }
  }
}

// Pair of blocks `pair` of round `round`: load its 2JB x 2JB subproblem,
// run one cyclic Jacobi sweep over its indices (round-robin over 2JB
// players: JB disjoint rotations per inner round, applied together), and
// write the accumulated unitary U (column-major, JM x JM) and whether any
// rotation was made.  Indices >= k are padding: zero rows and columns that
// never rotate.  S0, S1 and U: JM x JLD arrays in LDS.
//
// Bound by the chain of the 2JB - 1 dependent inner rounds: one workgroup per
// pair, a few dozen on the chip.  In an inner round 16 threads compute the
// rotations and publish them; then waves 0 - 3 update S in LDS, one 2 x 2
// block a thread, beside waves 4 - 7, which keep U in registers: a lane holds
// the two columns of its position in the tournament, and the columns move on
// by one lane after a round (U in LDS: 5% more at k = 260, its reads and
// writes hold up those of S).  The inner rounds are 20 of a launch's 27 us at
// k = 140 (complex; 10 us more with S and U updated in turn by the same four
// waves and a tangent-form rotation).  Slower: every thread computing its own
// rotations (3 us), which saves the exchange but repeats the square roots in
// all waves; reading the blocks of S before the rotations are known, by the
// same wave (4 us) or with the rotations in another (2 us): either way those
// reads come before the rotations' own.  Rotating only across the two blocks
// after a sweep's first round halves the inner rounds but takes 38% more
// sweeps.
template <class T>
__device__ void pair_body(const T* __restrict__ G, int64_t ldg, int k, int nb, int round,
                          int pair, double thr, T* __restrict__ ubuf, int* __restrict__ flags,
                          const T* __restrict__ uprev, T* S, T* U, T* Ts) {
  __shared__ double rcs[JB], rsn[JB];
  __shared__ T rph[JB];
  __shared__ int rrot[JB];
  __shared__ int any, turn;
  const int tid = threadIdx.x;
  const int bp = rr_player(nb, round, pair), bq = rr_player(nb, round, nb - 1 - pair);
  auto gidx = [&](int l) { return l < JB ? bp * JB + l : bq * JB + (l - JB); };
  if (tid == 0) any = 0;
  for (int e = tid; e < JM * JM; e += JPT) {
    const int r = e % JM, c = e / JM;
    const int gr = gidx(r), gc = gidx(c);
    if (round == 0) {
      T v = from_real<T>(0.0);
      if (gr < k && gc < k) v = G[gr + (int64_t)gc * ldg];
      S[c * JLD + r] = v;
    }
  }
  if (round > 0) pair_load<T>(G, ldg, k, nb, round - 1, bp, bq, uprev, S, Ts);
  __syncthreads();
  const int half = tid / JT, t = tid % JT;
  // S: pairs i (rows) and j (columns), consecutive lanes along the rows; U:
  // pair j's columns, in the lanes of a DPP row, at rows i and i + JB
  const int j = half ? t % JB : t / JB, i = half ? t / JB : t % JB;
  T ut[2], ub[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ut[h] = from_real<T>(j == i + h * JB ? 1.0 : 0.0);
    ub[h] = from_real<T>(JM - 1 - j == i + h * JB ? 1.0 : 0.0);
  }
  for (int rr = 0; rr < JM - 1; ++rr) {
    if (tid < JB) {
      const int a = inner_player(rr, tid), b = inner_player(rr, JM - 1 - tid);
      double cs, sn;
      T ph;
      const int rot = jac_rotation(real_(S[a * JLD + a]), real_(S[b * JLD + b]), S[b * JLD + a],
                                   thr, cs, sn, ph);
      rcs[tid] = cs;
      rsn[tid] = sn;
      rph[tid] = ph;
      rrot[tid] = rot;
      const bool some = __any(rot);
      if (tid == 0) {
        turn = some;
        if (some) any = 1;
      }
    }
    const int aj = inner_player(rr, j), bj = inner_player(rr, JM - 1 - j);
    const int ai = inner_player(rr, i), bi = inner_player(rr, JM - 1 - i);
    __syncthreads();
    if (turn) {  // the same in every thread
      const double cj = rcs[j], sj = rsn[j];
      const T pjc = conj_(rph[j]);
      if (half == 0) {
        // S <- u^H S u on the 2 x 2 block (rows of pair i, columns of pair j)
        const double ci = rcs[i], si = rsn[i];
        const T pi_ = rph[i];
        // u_i^H M u_j = R_i^T (D_i^H M D_j) R_j: phases first, then the real
        // rotations
        const T m00 = S[aj * JLD + ai];
        const T m01 = S[bj * JLD + ai] * pjc;
        const T m10 = pi_ * S[aj * JLD + bi];
        const T m11 = S[bj * JLD + bi] * (pi_ * pjc);
        const T r00 = m00 * cj - m01 * sj, r01 = m00 * sj + m01 * cj;
        const T r10 = m10 * cj - m11 * sj, r11 = m10 * sj + m11 * cj;
        T n00 = r00 * ci - r10 * si, n01 = r01 * ci - r11 * si;
        T n10 = r00 * si + r10 * ci, n11 = r01 * si + r11 * ci;
        if (i == j) {
          // the pivot block: exactly diagonal and real after its rotation
          n00 = from_real<T>(real_(n00));
          n11 = from_real<T>(real_(n11));
          if (rrot[i]) {
            n01 = from_real<T>(0.0);
            n10 = from_real<T>(0.0);
          }
        }
        S[aj * JLD + ai] = n00;
        S[bj * JLD + ai] = n01;
        S[aj * JLD + bi] = n10;
        S[bj * JLD + bi] = n11;
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const T u0 = ut[h], u1 = ub[h] * pjc;
          ut[h] = u0 * cj - u1 * sj;
          ub[h] = u0 * sj + u1 * cj;
        }
      }
    }
    if (half == 1) {
      // the players move on by one position: the first halves down, the
      // second up, position 0 stays
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const T nt = from_lane_above(ut[h]), nb_ = from_lane_below(ub[h]);
        const T t0 = ut[h], b0 = ub[h];
        ut[h] = pick(j == 0, t0, pick(j == JB - 1, b0, nt));
        ub[h] = pick(j == 0, nt, nb_);
      }
    }
    __syncthreads();
  }
  if (half == 1)  // 2 JB - 1 moves: every player is back
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      U[j * JLD + i + h * JB] = ut[h];
      U[(JM - 1 - j) * JLD + i + h * JB] = ub[h];
    }
  __syncthreads();
  // One Newton-Schulz step towards the nearest unitary, U <- U (3 I - U^H U) / 2:
  // the rounding of the rotations leaves U unitary only to a few ulps per
  // inner round, and applying a non-unitary J^H G J shifts the eigenvalues by
  // that much in every round; the step brings it back to rounding level.
  // M = U^H U goes into S (no longer needed).  Both products on the matrix
  // cores, a quadrant in each of four waves: with every thread summing its
  // entries from LDS they took 5 us of a launch.
  if (any) {
    const int lane = tid & 63, w = tid >> 6, l16 = lane & 15, lk = lane >> 4;
    const int i0 = JB * (w & 1), c0 = JB * (w >> 1);
    T a[JM / 4], b[JM / 4], out[4];
    if (w < 4) {
#pragma unroll
      for (int st = 0; st < JM / 4; ++st) {
        a[st] = conj_(U[(i0 + l16) * JLD + 4 * st + lk]);
        b[st] = U[(c0 + l16) * JLD + 4 * st + lk];
      }
      quad_mma(a, b, out);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(c0 + lk + 4 * q) * JLD + i0 + l16] = out[q];
    }
    __syncthreads();
    if (w < 4) {
#pragma unroll
      for (int st = 0; st < JM / 4; ++st) {
        a[st] = U[(4 * st + lk) * JLD + i0 + l16];
        b[st] = S[(c0 + l16) * JLD + 4 * st + lk];
      }
      quad_mma(a, b, out);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        out[q] = U[(c0 + lk + 4 * q) * JLD + i0 + l16] * 1.5 - out[q] * 0.5;
    }
    __syncthreads();
    if (w < 4)
#pragma unroll
      for (int q = 0; q < 4; ++q) U[(c0 + lk + 4 * q) * JLD + i0 + l16] = out[q];
    __syncthreads();
  }
  T* Uo = ubuf + (int64_t)pair * JM * JM;
  for (int e = tid; e < JM * JM; e += JPT) Uo[e] = U[(e / JM) * JLD + (e % JM)];
  if (tid == 0) flags[pair] = any;
}

// JM rows of V (row chunk `chunk`) times the columns of pair b of round
// `round`: V <- V U_b (nothing if the pair did not rotate).  Xs, Bs: LDS.
template <class T>
__device__ void vtile_body(T* __restrict__ V, int64_t ldv, int k, int nb, int round, int b,
                           int chunk, const T* __restrict__ ubuf, const int* __restrict__ flags,
                           T* Xs, T* Bs) {
  if (!flags[b]) return;
  const int tid = threadIdx.x;
  const int b0 = rr_player(nb, round, b), b1 = rr_player(nb, round, nb - 1 - b);
  auto gb = [&](int l) { return l < JB ? b0 * JB + l : b1 * JB + (l - JB); };
  const T* Ub = ubuf + (int64_t)b * JM * JM;
  const int64_t r0 = (int64_t)chunk * JM;
  for (int e = tid; e < JM * JM; e += JPT) {
    const int r = e % JM, c = e / JM;
    const int gc = gb(c);
    T v = from_real<T>(0.0);
    if (r0 + r < k && gc < k) v = V[r0 + r + (int64_t)gc * ldv];
    Xs[c * JLD + r] = v;
    Bs[r * JLD + c] = Ub[e];
  }
  __syncthreads();
  if (tid >= JT) return;  // four waves, one quadrant each
  T out[4];
  tile_mma(Xs, Bs, out);
  const int64_t row = r0 + mma_row();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int gc = gb(mma_col(r));
    if (row < k && gc < k) V[row + (int64_t)gc * ldv] = out[r];
  }
}

// Tile of the updated matrix at (pair a rows, pair b columns), a <= b, of
// round `round`: U_a^H X U_b, and its mirror (b, a) the conjugate transpose
// (a == b: the Hermitian part); copied where neither pair rotated.  All
// threads of the workgroup move data, four waves multiply.
template <class T>
__device__ void gtile_body(const T* __restrict__ G, int64_t ldg, T* __restrict__ D, int64_t ldd,
                           int k, int nb, int round, int t, const T* __restrict__ ubuf,
                           const int* __restrict__ flags, T* Xs, T* Bs, T* Ts) {
  // Xs: X(i, l) at Xs[l * JLD + i], later the result Y; Bs: U_b (B(l, c) at
  // Bs[l * JLD + c]), then A = U_a^H; Ts: X U_b, T(l, c) at Ts[l * JLD + c]
  const int tid = threadIdx.x;
  int b = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  if ((b + 1) * (b + 2) / 2 <= t) ++b;
  if (b * (b + 1) / 2 > t) --b;
  const int a = t - b * (b + 1) / 2;
  const int fa = flags[a], fb = flags[b];
  const int a0 = rr_player(nb, round, a), a1 = rr_player(nb, round, nb - 1 - a);
  const int b0 = rr_player(nb, round, b), b1 = rr_player(nb, round, nb - 1 - b);
  auto ga = [&](int l) { return l < JB ? a0 * JB + l : a1 * JB + (l - JB); };
  auto gb = [&](int l) { return l < JB ? b0 * JB + l : b1 * JB + (l - JB); };
  const T* Ua = ubuf + (int64_t)a * JM * JM;
  const T* Ub = ubuf + (int64_t)b * JM * JM;
  const bool rot = fa || fb;
  for (int e = tid; e < JM * JM; e += JPT) {
    const int r = e % JM, c = e / JM;
    const int gr = ga(r), gc = gb(c);
    T v = from_real<T>(0.0);
    if (gr < k && gc < k) v = G[gr + (int64_t)gc * ldg];
    Xs[c * JLD + r] = v;
    if (rot) Bs[r * JLD + c] = fb ? Ub[e] : from_real<T>(r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  if (rot) {
    T out[4];
    if (tid < JT) {
      tile_mma(Xs, Bs, out);  // T = X U_b
#pragma unroll
      for (int r = 0; r < 4; ++r) Ts[mma_row() * JLD + mma_col(r)] = out[r];
    }
    __syncthreads();
    // A(c, r) = conj(U_a(r, c)) at Bs[r * JLD + c]
    for (int e = tid; e < JM * JM; e += JPT) {
      const int r = e % JM, c = e / JM;
      Bs[r * JLD + c] = fa ? conj_(Ua[e]) : from_real<T>(r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (tid < JT) {
      tile_mma(Bs, Ts, out);  // Y = U_a^H T, stored as Y(i, c) at Xs[c * JLD + i]
#pragma unroll
      for (int r = 0; r < 4; ++r) Xs[mma_col(r) * JLD + mma_row()] = out[r];
    }
    __syncthreads();
  }
  const int i = tid % JM, gi = ga(i), gm = gb(i);
#pragma unroll
  for (int c = tid / JM; c < JM; c += JPT / JM) {
    const int gc = gb(c), gt = ga(c);
    if (a == b) {
      T v = (Xs[c * JLD + i] + conj_(Xs[i * JLD + c])) * 0.5;
      if (i == c) v = from_real<T>(real_(v));
      if (gi < k && gc < k) D[gi + (int64_t)gc * ldd] = v;
    } else {
      if (gi < k && gc < k) D[gi + (int64_t)gc * ldd] = Xs[c * JLD + i];
      // mirror: lanes run over the rows of the (b, a) tile
      if (gm < k && gt < k) D[gm + (int64_t)gt * ldd] = conj_(Xs[i * JLD + c]);
    }
  }
}

// One round of a sweep, one launch.  Workgroups [0, npairs) solve the pairs
// of round `round` into (ubuf, flags), each forming its own subproblem from
// the matrix G before round - 1 and that round's unitaries (uprev, fprev);
// beside them the next `gtiles` apply those unitaries to the whole matrix, G
// -> D, and the rest to the eigenvector block.  Nothing a workgroup writes
// is read in the same launch.
//
// A launch of pairs and eigenvectors followed by one of the matrix in place
// leaves the second's time and a launch gap on the chain of the rounds: 32.4
// + gap against 27.3 us a round at k = 140, 42 against 34 at k = 260 (complex;
// 33 and 41 before the Newton-Schulz step moved to the matrix cores).  A
// dense matrix, complex: k = 140 3.17 -> 2.66 ms, 256 5.9 -> 4.93, 700 21.9 ->
// 18.6; the copied tiles and the 60 KB of LDS cost less than the launch at
// every order measured, to 1300.
template <class T>
__global__ __launch_bounds__(JPT) void jac_round_k(
    const T* __restrict__ G, int64_t ldg, T* __restrict__ D, int64_t ldd, T* __restrict__ V,
    int64_t ldv, int k, int nb, int round, int npairs, int gtiles, double thr,
    T* __restrict__ ubuf, int* __restrict__ flags, const T* __restrict__ uprev,
    const int* __restrict__ fprev) {
  __shared__ T sm0[JM * JLD];
  __shared__ T sm1[JM * JLD];
  __shared__ T sm2[3 * JM * THLD];
  static_assert(3 * JM * THLD >= JM * JLD, "tile of gtile_body");
  const int w = blockIdx.x;
  if (w < npairs) {
    pair_body<T>(G, ldg, k, nb, round, w, thr, ubuf, flags, uprev, sm0, sm1, sm2);
  } else if (w < npairs + gtiles) {
    gtile_body<T>(G, ldg, D, ldd, k, nb, round - 1, w - npairs, uprev, fprev, sm0, sm1, sm2);
  } else {
    const int P = nb / 2, t = w - npairs - gtiles;
    vtile_body<T>(V, ldv, k, nb, round - 1, t % P, t / P, uprev, fprev, sm0, sm1);
  }
}

// part[2 w] = sum of |G_ij|^2 off the diagonal, part[2 w + 1] on it, over
// the entries workgroup w visits.
template <class T>
__global__ __launch_bounds__(JT) void jac_norms_k(const T* __restrict__ G, int64_t ldg, int k,
                                                  double* __restrict__ part) {
  __shared__ double so[JT], sd[JT];
  double off = 0.0, dia = 0.0;
  const int64_t total = (int64_t)k * k;
  for (int64_t e = (int64_t)blockIdx.x * JT + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * JT) {
    const int64_t r = e % k, c = e / k;
    const double v = abs2(G[r + c * ldg]);
    if (r == c)
      dia += v;
    else
      off += v;
  }
  so[threadIdx.x] = off;
  sd[threadIdx.x] = dia;
  __syncthreads();
  for (int s = JT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      so[threadIdx.x] += so[threadIdx.x + s];
      sd[threadIdx.x] += sd[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = so[0];
    part[2 * blockIdx.x + 1] = sd[0];
  }
}

// Sort of the k values w: thread j counts those that come before w[j] (ties
// and NaN, taken as the largest, in index order), which is its place.
__global__ __launch_bounds__(JT) void jac_sort_k(const double* __restrict__ w, int k,
                                                 double* __restrict__ sorted,
                                                 int* __restrict__ perm) {
  __shared__ double tile[JT];
  const int j = blockIdx.x * JT + threadIdx.x;
  auto key = [](double x) { return x == x ? x : INFINITY; };
  const double wj = j < k ? w[j] : 0.0, kj = key(wj);
  int rank = 0;
  for (int i0 = 0; i0 < k; i0 += JT) {
    __syncthreads();
    if (i0 + (int)threadIdx.x < k) tile[threadIdx.x] = key(w[i0 + threadIdx.x]);
    __syncthreads();
    const int m = min(JT, k - i0);
    for (int i = 0; i < m; ++i) rank += tile[i] < kj || (tile[i] == kj && i0 + i < j);
  }
  if (j < k) {
    sorted[rank] = wj;
    perm[rank] = j;
  }
}

template <class T>
__global__ void jac_eye_k(T* __restrict__ V, int64_t ldv, int k) {
  const int64_t total = (int64_t)k * k;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e % k, c = e / k;
    V[r + c * ldv] = from_real<T>(r == c ? 1.0 : 0.0);
  }
}

inline int jac_blocks(int k) {
  int nb = (k + JB - 1) / JB;
  if (nb < 2) nb = 2;
  return nb + (nb & 1);
}

// Workspace layout for orders up to kmax (byte offsets): the pairs' unitaries
// and rotation flags of two rounds, the diagonal.
struct JacLayout {
  size_t ubuf[2], flags[2], diag, total;
  JacLayout(bool cplx, int kmax) {
    const int P = jac_blocks(std::max(kmax, 1)) / 2;
    const size_t esz = cplx ? 16 : 8;
    const size_t ub = ((size_t)P * JM * JM * esz + 255) / 256 * 256;
    const size_t fl = ((size_t)P * 4 + 255) / 256 * 256;
    ubuf[0] = 0;
    ubuf[1] = ub;
    flags[0] = 2 * ub;
    flags[1] = 2 * ub + fl;
    diag = 2 * ub + 2 * fl;
    total = diag + (size_t)std::max(kmax, 1) * 8;
  }
};

template <class T>
struct JacobiRunner {
  // the partial sums go straight to host memory
  static void norms(const void* G, int64_t ldg, int k, double* pinned, double* off2,
                    double* dia2, hipStream_t st) {
    hipLaunchKernelGGL(jac_norms_k<T>, dim3(NPART), dim3(JT), 0, st, static_cast<const T*>(G),
                       ldg, k, pinned);
    CHASE_HIP(hipGetLastError());
    CHASE_HIP(hipStreamSynchronize(st));
    double o = 0.0, d = 0.0;
    for (int w = 0; w < NPART; ++w) {
      o += pinned[2 * w];
      d += pinned[2 * w + 1];
    }
    *off2 = o;
    *dia2 = d;
  }

  static int run(void* G, int64_t ldg, int k, void* V, int64_t ldv, void* ws, void* G2,
                 const JacLayout& lay, double* pinned, double tol, int max_sweeps, double off2,
                 double dia2, hipStream_t st) {
    const int nb = jac_blocks(k), P = nb / 2;
    char* base = static_cast<char*>(ws);
    T* ubuf[2] = {reinterpret_cast<T*>(base + lay.ubuf[0]), reinterpret_cast<T*>(base + lay.ubuf[1])};
    int* flags[2] = {reinterpret_cast<int*>(base + lay.flags[0]),
                     reinterpret_cast<int*>(base + lay.flags[1])};
    const int tiles_g = P * (P + 1) / 2;
    const int tiles_v = ((k + JM - 1) / JM) * P;
    // the matrix and its other buffer, exchanged by every round's update
    T *Gt = static_cast<T*>(G), *Do = static_cast<T*>(G2);
    int64_t ldt = ldg, ldo = k;
    T* Vt = static_cast<T*>(V);
    hipLaunchKernelGGL(jac_eye_k<T>, dim3(std::min<int64_t>(1024, ((int64_t)k * k + 255) / 256)),
                       dim3(256), 0, st, Vt, ldv, k);
    CHASE_HIP(hipGetLastError());
    const double fro2 = off2 + dia2;
    const double thr = tol * std::sqrt(fro2) / (double)k;
    int sweeps = 0;
    while (!(off2 <= tol * tol * fro2)) {
      if (sweeps >= max_sweeps)
        throw Error(CHASE_ERR_NUMERIC, "Jacobi eigensolver did not converge in " +
                                           std::to_string(max_sweeps) + " sweeps");
      // round r: its pairs, with the matrix and eigenvector updates of r - 1;
      // the last round's updates close the sweep
      for (int r = 0; r <= nb - 1; ++r) {
        const int np = r < nb - 1 ? P : 0, cur = r & 1, prev = (r + 1) & 1;
        const int ng = r > 0 ? tiles_g : 0, nv = r > 0 ? tiles_v : 0;
        hipLaunchKernelGGL(jac_round_k<T>, dim3(np + ng + nv), dim3(JPT), 0, st,
                           static_cast<const T*>(Gt), ldt, Do, ldo, Vt, ldv, k, nb, r, np, ng,
                           thr, ubuf[cur], flags[cur], static_cast<const T*>(ubuf[prev]),
                           static_cast<const int*>(flags[prev]));
        if (r > 0) {
          std::swap(Gt, Do);
          std::swap(ldt, ldo);
        }
      }
      CHASE_HIP(hipGetLastError());
      ++sweeps;
      double d2;
      norms(Gt, ldt, k, pinned, &off2, &d2, st);
      if (!std::isfinite(off2)) throw Error(CHASE_ERR_NUMERIC, "non-finite entries in Jacobi");
    }
    diag_real(sizeof(T) == 16, Gt, ldt, k, reinterpret_cast<double*>(base + lay.diag), st);
    return sweeps;
  }
};

}  // namespace

size_t jacobi_ws_bytes(bool cplx, int kmax) { return JacLayout(cplx, kmax).total; }

void jacobi_norms(bool cplx, const void* G, int64_t ldg, int k, double* pinned, double* off2,
                  double* dia2, hipStream_t st) {
  CHASE_REQUIRE(k >= 1, "Jacobi eigensolver: order out of range");
  static_assert(kJacobiPinned >= 2 * NPART, "pinned partial sums");
  if (cplx)
    JacobiRunner<cd>::norms(G, ldg, k, pinned, off2, dia2, st);
  else
    JacobiRunner<double>::norms(G, ldg, k, pinned, off2, dia2, st);
}

int jacobi_heev(bool cplx, void* G, int64_t ldg, int k, void* V, int64_t ldv, void* W,
                int64_t ldw, double* d_evals, int* d_perm, void* ws, int kmax, void* G2,
                double* pinned, hipStream_t st, double off2, double dia2, double tol, int max_sweeps) {
  CHASE_REQUIRE(k >= 1 && k <= kmax, "Jacobi eigensolver: order out of range");
  CHASE_REQUIRE(ldg >= k && ldv >= k && ldw >= k, "Jacobi eigensolver: leading dimension < k");
  CHASE_REQUIRE(V != G && V != W, "Jacobi eigensolver: V must be a separate buffer");
  CHASE_REQUIRE(G2 != G && G2 != V && G2 != W, "Jacobi eigensolver: G2 must be a separate buffer");
  if (!std::isfinite(off2) || !std::isfinite(dia2))
    throw Error(CHASE_ERR_NUMERIC, "non-finite entries in the projected matrix");
  const JacLayout lay(cplx, kmax);
  int sweeps;
  if (cplx)
    sweeps = JacobiRunner<cd>::run(G, ldg, k, V, ldv, ws, G2, lay, pinned, tol, max_sweeps, off2, dia2,
                                   st);
  else
    sweeps = JacobiRunner<double>::run(G, ldg, k, V, ldv, ws, G2, lay, pinned, tol, max_sweeps, off2,
                                       dia2, st);
  // eigenvalues: the diagonal, ascending (stable), eigenvectors gathered to match
  double* d_diag = reinterpret_cast<double*>(static_cast<char*>(ws) + lay.diag);
  hipLaunchKernelGGL(jac_sort_k, dim3((unsigned)((k + JT - 1) / JT)), dim3(JT), 0, st, d_diag, k,
                     d_evals, d_perm);
  CHASE_HIP(hipGetLastError());
  gather_cols(cplx, V, ldv, W, ldw, k, k, d_perm, st);
  return sweeps;
}

}  // namespace chase
