// Cholesky factorisation A = R^H R of the Gram matrix in the QR step's
// Cholesky passes (Algorithm 1's QR step, done as Cholesky QR with a shifted
// pass and a Householder fallback; the paper's own QR is geqrf, Section
// 2.3).  R is upper triangular with a positive real diagonal.
//
// Right-looking blocked algorithm with panels of CB rows.  Per panel two
// launches:
//  - chol_panel_k: every workgroup factors the CB x CB diagonal block in
//    LDS (the same arithmetic in each, so they agree bit for bit), then
//    solves R11^H X = A12 for its own PC columns of the row panel, staged
//    through LDS, each column held in the registers of a quad of lanes (forward
//    substitution).  The last workgroup to have read the block stores R11.
//  - chol_update_k: A22 -= R12^H R12 on the upper triangle, in UT x UT
//    tiles staged through LDS.
// The order of a k x k factorisation is about k / CB panel steps; at the
// sizes of the subspace (k ~ 10^3) each launch is short and the chain is
// latency bound, which the one-launch panel keeps to two launches a panel.
//
// A pivot that is not positive (or not a number) stops the factorisation:
// info receives its 1-based order (as LAPACK's potrf) and every later
// launch returns at once; R then holds partial results.
#include "common.h"

#include <algorithm>
#include <utility>

namespace chase {
namespace {

constexpr int CB = 32;        // panel rows
constexpr int CLD = CB + 1;   // LDS leading dimension of the diagonal block
constexpr int CT = 256;       // threads per workgroup
constexpr int CG = CT / CB;   // column groups of the (row, column-group) thread map
constexpr int PQ = 4;         // threads per row-panel column (one quad of lanes)
constexpr int PC = CT / PQ;   // row-panel columns per workgroup
constexpr int PLD = PC + 1;
constexpr int UT = 32;        // trailing-update tile
constexpr int ULD = UT + 1;

struct cd {
  double x, y;
};
__device__ __forceinline__ cd operator-(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cd operator*(cd a, double s) { return {a.x * s, a.y * s}; }
__device__ __forceinline__ double real_(double a) { return a; }
__device__ __forceinline__ double real_(cd a) { return a.x; }
__device__ __forceinline__ double scaled(double a, double s) { return a * s; }
__device__ __forceinline__ cd scaled(cd a, double s) { return a * s; }
template <class T>
__device__ __forceinline__ T from_real(double a);
template <>
__device__ __forceinline__ double from_real<double>(double a) { return a; }
template <>
__device__ __forceinline__ cd from_real<cd>(double a) { return {a, 0.0}; }
// acc -= conj(a) * b
__device__ __forceinline__ void msub_conj(double& acc, double a, double b) {
  acc = fma(-a, b, acc);
}
__device__ __forceinline__ void msub_conj(cd& acc, cd a, cd b) {
  acc.x = fma(-a.x, b.x, acc.x);
  acc.x = fma(-a.y, b.y, acc.x);
  acc.y = fma(-a.x, b.y, acc.y);
  acc.y = fma(a.y, b.x, acc.y);
}
// acc += conj(a) * b
__device__ __forceinline__ void mac_conj(double& acc, double a, double b) { acc = fma(a, b, acc); }
__device__ __forceinline__ void mac_conj(cd& acc, cd a, cd b) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(-a.y, b.x, acc.y);
}

// acc -= a * b
__device__ __forceinline__ void msub(double& acc, double a, double b) { acc = fma(-a, b, acc); }
__device__ __forceinline__ void msub(cd& acc, cd a, cd b) {
  acc.x = fma(-a.x, b.x, acc.x);
  acc.x = fma(a.y, b.y, acc.x);
  acc.y = fma(-a.x, b.y, acc.y);
  acc.y = fma(-a.y, b.x, acc.y);
}
// Value of lane l of each group of `width` lanes.
__device__ __forceinline__ double lane_bcast(double a, int l, int width) {
  return __shfl(a, l, width);
}
__device__ __forceinline__ cd lane_bcast(cd a, int l, int width) {
  return {__shfl(a.x, l, width), __shfl(a.y, l, width)};
}

// Value of lane Q of each quad of lanes.
template <int Q>
__device__ __forceinline__ double quad_bcast(double a) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(a), Q * 0x55, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(a), Q * 0x55, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int Q>
__device__ __forceinline__ cd quad_bcast(cd a) {
  return {quad_bcast<Q>(a.x), quad_bcast<Q>(a.y)};
}

// Step L of the row panel's substitution: row L is final after its scaling;
// the rows below take conj(R11(L, i)) x_L off.
template <class T, int L>
__device__ __forceinline__ void solve_row(T (&x)[CB / PQ], const T* D, const double* rdg, int q) {
  constexpr int M = L / PQ, Q = L % PQ;
  const T xs = scaled(x[M], rdg[L]);
  if (q == Q) x[M] = xs;
  const T xl = quad_bcast<Q>(xs);
#pragma unroll
  for (int m = M; m < CB / PQ; ++m) {
    const int i = m * PQ + q;
    if (m > M || q > Q) msub_conj(x[m], D[L + i * CLD], xl);
  }
}
template <class T, int... L>
__device__ __forceinline__ void solve_rows(T (&x)[CB / PQ], const T* D, const double* rdg, int q,
                                           std::integer_sequence<int, L...>) {
  (solve_row<T, L>(x, D, rdg, q), ...);
}

// Panel j0: factor the diagonal block and solve the row panel.  Grid:
// ceil((k - j0 - CB) / PC) workgroups (at least one).  Thread (ti, tg) =
// (tid % CB, tid / CB) owns row ti of the diagonal block at the columns
// tg + CG q (q < CB / CG), in registers.
template <class T>
__global__ __launch_bounds__(CT) void chol_panel_k(T* __restrict__ A, int64_t lda, int k, int j0,
                                                   int* __restrict__ info) {
  constexpr int NQ = CB / CG;
  __shared__ T D[CB * CLD];    // R11, column-major: D[i + c * CLD]
  __shared__ T P[CB * PLD];    // this workgroup's row-panel columns: P[i * PLD + c]
  __shared__ T row[2][CB];     // the pivot row of the current and the next step
  __shared__ double piv[CB];   // pivots a_jj = r_jj^2
  __shared__ double rdg[CB];   // 1 / r_jj
  __shared__ int last;         // this workgroup stores R11
  const int bad = *info;       // loaded with the tiles below, tested after them
  const int tid = threadIdx.x;
  const int ti = tid % CB, tg = tid / CB;
  const int nb = min(CB, k - j0);
  // only full panels have columns to the right (nb < CB means j0 + nb == k)
  const int64_t c0 = (int64_t)j0 + nb + (int64_t)blockIdx.x * PC;
  const int pc = nb == CB ? (int)max<int64_t>(0, min<int64_t>(PC, k - c0)) : 0;
  T v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int c = tg + CG * q;
    v[q] = (ti <= c && c < nb) ? A[(int64_t)(j0 + ti) + (int64_t)(j0 + c) * lda]
                               : from_real<T>(0.0);
  }
  for (int c = tg; c < pc; c += CG) P[ti * PLD + c] = A[(int64_t)(j0 + ti) + (c0 + c) * lda];
  if (bad != 0) return;
  if (ti == 0)
#pragma unroll
    for (int q = 0; q < NQ; ++q) row[0][tg + CG * q] = v[q];
  __syncthreads();
  // Unscaled right-looking elimination: step j takes conj(a_ji) a_jc / a_jj
  // off every a_ic, j < i <= c, and the owners of row j + 1 (final after
  // this step) publish it for the next step.  Row j ends as r_jj * (row j
  // of R) with a_jj = r_jj^2.
  for (int j = 0; j < nb; ++j) {
    const T* rj = row[j & 1];
    const double d = real_(rj[j]);
    if (!(d > 0.0)) {  // the same value in every thread: a uniform exit
      if (tid == 0 && blockIdx.x == 0) *info = j0 + j + 1;
      return;
    }
    if (tid == 0) piv[j] = d;
    if (ti > j && ti < nb) {
      const T f = scaled(rj[ti], 1.0 / d);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int c = tg + CG * q;
        if (c >= ti && c < nb) msub_conj(v[q], f, rj[c]);
      }
      if (ti == j + 1)
#pragma unroll
        for (int q = 0; q < NQ; ++q) row[(j + 1) & 1][tg + CG * q] = v[q];
    }
    __syncthreads();
  }
  if (ti < nb) {
    const double r = sqrt(piv[ti]);
    const double rs = 1.0 / r;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = tg + CG * q;
      if (c > ti && c < nb) D[ti + c * CLD] = scaled(v[q], rs);
      if (c == ti) D[ti + c * CLD] = from_real<T>(r);
    }
    if (tg == 0) rdg[ti] = rs;
  }
  __syncthreads();
  // The factor takes the diagonal block's place once every workgroup has read the
  // block (all of its entries went into D by now): the one that counts last, in
  // info[1], stores it.  Workgroup 0 storing it here could be ahead of one that
  // has not begun, on a busy chip or with more workgroups than the chip holds.
  int before = 0;
  if (tid == 0 && gridDim.x > 1) before = atomicAdd(info + 1, 1);
  auto store_factor = [&] {
    if (ti < nb)
      for (int c = tg; c < nb; c += CG)
        if (ti <= c) A[(int64_t)(j0 + ti) + (int64_t)(j0 + c) * lda] = D[ti + c * CLD];
  };
  // Row panel: column c of A12 becomes R11^{-H} a_c (forward substitution,
  // column-oriented, in registers).  Lane q of a column's quad holds its rows q,
  // q + 4, ...; the finished row goes to the other three by a quad broadcast.
  // One thread per column spent 11 us on the 496 multiply-adds and factor reads
  // of a column, the longest phase of the launch; a quad 3 us.  The last panel has
  // none, and one workgroup.
  if (pc == 0) {
    store_factor();
    return;
  }
  {
    const int c = tid / PQ, q = tid % PQ;
    T x[CB / PQ];
    if (c < pc) {
#pragma unroll
      for (int m = 0; m < CB / PQ; ++m) x[m] = P[(m * PQ + q) * PLD + c];
    } else {
#pragma unroll
      for (int m = 0; m < CB / PQ; ++m) x[m] = from_real<T>(0.0);
    }
    solve_rows<T>(x, D, rdg, q, std::make_integer_sequence<int, CB>{});
    if (c < pc) {
#pragma unroll
      for (int m = 0; m < CB / PQ; ++m) P[(m * PQ + q) * PLD + c] = x[m];
    }
  }
  if (tid == 0) {
    last = before == (int)gridDim.x - 1;
    if (last && gridDim.x > 1) info[1] = 0;  // for the next panel
  }
  __syncthreads();
  if (last) store_factor();
  for (int c = tg; c < pc; c += CG) A[(int64_t)(j0 + ti) + (c0 + c) * lda] = P[ti * PLD + c];
}

// A22 -= R12^H R12 on the upper triangle of the trailing block (rows and
// columns from j0 + CB), R12 in rows j0 .. j0 + CB - 1.  Grid t x t with
// t = ceil(m / UT); workgroups below the diagonal return.
template <class T>
__global__ __launch_bounds__(CT) void chol_update_k(T* __restrict__ A, int64_t lda, int k, int j0,
                                                    const int* __restrict__ info) {
  __shared__ T Ri[CB * ULD];  // Ri[l * ULD + q] = R12(l, i0 + q)
  __shared__ T Rc[CB * ULD];
  const int ti = blockIdx.x, tc = blockIdx.y;
  if (ti > tc || *info != 0) return;
  const int tid = threadIdx.x;
  const int b = j0 + CB;  // first row and column of the trailing block
  const int m = k - b;
  const int i0 = ti * UT, c0 = tc * UT;
  const int ni = min(UT, m - i0), nc = min(UT, m - c0);
  for (int e = tid; e < CB * UT; e += CT) {
    const int l = e % CB, q = e / CB;
    const T* row = A + (int64_t)(j0 + l);
    T vi = from_real<T>(0.0), vc = from_real<T>(0.0);
    if (q < ni) vi = row[(int64_t)(b + i0 + q) * lda];
    if (q < nc) vc = row[(int64_t)(b + c0 + q) * lda];
    Ri[l * ULD + q] = vi;
    Rc[l * ULD + q] = vc;
  }
  __syncthreads();
  const int ii = tid % UT;
  const int cg = tid / UT;  // column group
  constexpr int NG = CT / UT;
  constexpr int PER = UT / NG;
  T acc[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) acc[p] = from_real<T>(0.0);
#pragma unroll 4
  for (int l = 0; l < CB; ++l) {
    const T a = Ri[l * ULD + ii];
#pragma unroll
    for (int p = 0; p < PER; ++p) mac_conj(acc[p], a, Rc[l * ULD + cg + p * NG]);
  }
  if (ii >= ni) return;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int cc = cg + p * NG;
    if (cc >= nc || (ti == tc && ii > cc)) continue;
    T* dst = A + (int64_t)(b + i0 + ii) + (int64_t)(b + c0 + cc) * lda;
    *dst = *dst - acc[p];
  }
}

// M = diag(d) R^{-1} for an upper triangular R of order k <= IR * CT, zeros
// below the diagonal.  A workgroup solves R X = E for IC columns: from the
// last row panel that they reach up to the first, 32 rows at a time, the
// panel's triangle by back substitution in LDS, then its contribution taken off
// the rows above, which the threads hold in registers (thread t: rows t, t +
// CT).  Bound by the chain of k / 32 panels of 32 dependent steps; one launch
// where a library inverse takes eight and more (complex: 47 us against about 130
// with their gaps at k = 140, 214 against 319 at k = 512, the largest order the
// registers hold).
constexpr int IC = 4;  // columns per workgroup
constexpr int IR = 2;  // rows per thread

template <class T>
__global__ __launch_bounds__(CT) void chol_inverse_k(const T* __restrict__ R, int64_t ldr, int k,
                                                     const double* __restrict__ d,
                                                     T* __restrict__ M, int64_t ldm) {
  __shared__ T D[CB * CLD];     // the panel's triangle: D[i + c * CLD]
  __shared__ T Y[CB][IC];       // the panel's right-hand sides, then its solution
  __shared__ double rdg[CB];    // 1 / r_ii
  const int tid = threadIdx.x;
  const int c0 = blockIdx.x * IC;
  const int jl = min(c0 + IC, k) - 1;  // last column
  T acc[IR][IC];
#pragma unroll
  for (int m = 0; m < IR; ++m)
#pragma unroll
    for (int c = 0; c < IC; ++c) acc[m][c] = from_real<T>(tid + m * CT == c0 + c ? 1.0 : 0.0);
  for (int p = jl / CB; p >= 0; --p) {
    const int r0 = p * CB, nb = min(CB, k - r0);
    // triangle and right-hand sides of the panel
    for (int e = tid; e < CB * CB; e += CT) {
      const int i = e % CB, c = e / CB;
      if (i <= c && c < nb) D[i + c * CLD] = R[(r0 + i) + (int64_t)(r0 + c) * ldr];
    }
    if (tid < nb) rdg[tid] = 1.0 / real_(R[(r0 + tid) + (int64_t)(r0 + tid) * ldr]);
#pragma unroll
    for (int m = 0; m < IR; ++m) {
      const int i = tid + m * CT - r0;
      if (i >= 0 && i < nb)
#pragma unroll
        for (int c = 0; c < IC; ++c) Y[i][c] = acc[m][c];
    }
    __syncthreads();
    // back substitution: thread (c, i) of the first CB * IC holds entry (i, c)
    if (tid < CB * IC) {
      const int c = tid / CB, i = tid % CB;  // a column is half a wave
      T y = i < nb ? Y[i][c] : from_real<T>(0.0);
      for (int l = nb - 1; l >= 0; --l) {
        const T xl = lane_bcast(scaled(y, rdg[l]), l, CB);
        if (i == l) y = xl;
        if (i < l) msub(y, D[i + l * CLD], xl);
      }
      if (i < nb) Y[i][c] = y;
    }
    __syncthreads();
    // rows above: acc -= R(row, panel) Y; rows of the panel: the solution
#pragma unroll
    for (int m = 0; m < IR; ++m) {
      const int row = tid + m * CT;
      if (row < r0) {
        for (int l = 0; l < nb; ++l) {
          const T a = R[row + (int64_t)(r0 + l) * ldr];
#pragma unroll
          for (int c = 0; c < IC; ++c) msub(acc[m][c], a, Y[l][c]);
        }
      } else if (row < r0 + nb) {
#pragma unroll
        for (int c = 0; c < IC; ++c) acc[m][c] = Y[row - r0][c];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < IR; ++m) {
    const int row = tid + m * CT;
    if (row >= k) continue;
#pragma unroll
    for (int c = 0; c < IC; ++c)
      if (c0 + c < k)
        M[row + (int64_t)(c0 + c) * ldm] =
            row <= c0 + c ? scaled(acc[m][c], d[row]) : from_real<T>(0.0);
  }
}

template <class T>
void cholesky_launch(T* A, int64_t lda, int k, int* info, hipStream_t st) {
  for (int j0 = 0; j0 < k; j0 += CB) {
    const int nb = std::min(CB, k - j0);
    const int m = k - j0 - nb;
    const unsigned gp = (unsigned)std::max(1, (m + PC - 1) / PC);
    hipLaunchKernelGGL(chol_panel_k<T>, dim3(gp), dim3(CT), 0, st, A, lda, k, j0, info);
    CHASE_HIP(hipGetLastError());
    if (m > 0) {
      const unsigned t = (unsigned)((m + UT - 1) / UT);
      hipLaunchKernelGGL(chol_update_k<T>, dim3(t, t), dim3(CT), 0, st, A, lda, k, j0, info);
      CHASE_HIP(hipGetLastError());
    }
  }
}

}  // namespace

void cholesky_upper(bool cplx, void* A, int64_t lda, int k, int* d_info, hipStream_t st) {
  CHASE_REQUIRE(k >= 0 && lda >= std::max(1, k), "Cholesky: bad order or leading dimension");
  fill_zero(d_info, 2 * sizeof(int), st);
  if (k == 0) return;
  if (cplx)
    cholesky_launch(static_cast<cd*>(A), lda, k, d_info, st);
  else
    cholesky_launch(static_cast<double*>(A), lda, k, d_info, st);
}

bool chol_inverse(bool cplx, const void* R, int64_t ldr, int k, const double* d, void* M,
                  int64_t ldm, hipStream_t st) {
  if (k > IR * CT) return false;
  const dim3 grid((unsigned)((k + IC - 1) / IC));
  if (cplx)
    hipLaunchKernelGGL(chol_inverse_k<cd>, grid, dim3(CT), 0, st, static_cast<const cd*>(R), ldr, k,
                       d, static_cast<cd*>(M), ldm);
  else
    hipLaunchKernelGGL(chol_inverse_k<double>, grid, dim3(CT), 0, st,
                       static_cast<const double*>(R), ldr, k, d, static_cast<double*>(M), ldm);
  CHASE_HIP(hipGetLastError());
  return true;
}

}  // namespace chase
