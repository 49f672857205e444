// Host-side scalar logic of Algorithm 1: the Lanczos bound estimates (small
// tridiagonal eigenproblems and the density-of-states quadrature), the
// Chebyshev coefficients, the degree formula and the locking / sorting
// bookkeeping.  Plain C++ on arrays of at most nev+nex entries.
#include "hostmath.h"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace chase {

// Eigenvalues (ascending) of the real symmetric tridiagonal matrix with
// diagonal d and off-diagonal e, and the first component of each normalised
// eigenvector: the nodes and (squared) weights of the quadrature rule that a
// Lanczos run defines (Golub and Welsch, 1969).  Implicit QR steps with
// Wilkinson's shift (Golub & Van Loan, Section 8.3), the rotations applied to
// the first row of the eigenvector matrix only: O(k^2) for the whole problem
// (Jacobi sweeps over the dense k x k form took 1.7 ms a run at k = 25).
void tridiag_nodes(std::vector<double> d, std::vector<double> e, std::vector<double>& val,
                   std::vector<double>& first) {
  const int k = (int)d.size();
  std::vector<double> w(k, 0.0);
  if (k > 0) w[0] = 1.0;
  // a power of two brings the largest entry to [1, 2): squares below neither
  // overflow nor lose anything that matters
  double big = 0.0;
  for (int i = 0; i < k; ++i) {
    big = std::max(big, std::fabs(d[i]));
    if (i + 1 < k) big = std::max(big, std::fabs(e[i]));
  }
  const int ex = big > 0.0 && std::isfinite(big) ? std::ilogb(big) : 0;
  for (int i = 0; i < k; ++i) {
    d[i] = std::ldexp(d[i], -ex);
    e[i] = std::ldexp(e[i], -ex);
  }
  int hi = k - 1;
  for (int left = 100 * k; hi > 0 && left > 0; --left) {
    // the unreduced block [lo, hi] at the end of the matrix
    auto small = [&](int i) {
      return std::fabs(e[i]) <= 0x1p-53 * (std::fabs(d[i]) + std::fabs(d[i + 1])) + 0x1p-500;
    };
    if (small(hi - 1)) {
      --hi;
      continue;
    }
    int lo = hi - 1;
    while (lo > 0 && !small(lo - 1)) --lo;
    // shift: the eigenvalue of the last 2 x 2 block nearer to its last entry
    const double h = 0.5 * (d[hi - 1] - d[hi]), b = e[hi - 1];
    const double mu = d[hi] - b * (b / (h + std::copysign(std::sqrt(h * h + b * b), h)));
    double x = d[lo] - mu, z = e[lo];
    for (int i = lo; i < hi; ++i) {
      const double r = std::sqrt(x * x + z * z);
      const double c = r > 0.0 ? x / r : 1.0, s = r > 0.0 ? z / r : 0.0;
      if (i > lo) e[i - 1] = r;
      const double di = d[i], dj = d[i + 1], ei = e[i];
      const double p = s * (s * (dj - di) + 2.0 * c * ei);
      d[i] = di + p;
      d[i + 1] = dj - p;
      e[i] = c * s * (dj - di) + (c * c - s * s) * ei;
      if (i + 1 < hi) {
        x = e[i];
        z = s * e[i + 1];
        e[i + 1] *= c;
      }
      const double wi = w[i], wj = w[i + 1];
      w[i] = c * wi + s * wj;
      w[i + 1] = c * wj - s * wi;
    }
  }
  std::vector<int> idx(k);
  std::iota(idx.begin(), idx.end(), 0);
  std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return d[a] < d[b]; });
  val.resize(k);
  first.resize(k);
  for (int j = 0; j < k; ++j) {
    val[j] = std::ldexp(d[idx[j]], ex);
    first[j] = w[idx[j]];
  }
}

Bounds lanczos_bounds(const std::vector<double>& alpha, const std::vector<double>& beta, int nv,
                      int steps, int64_t n, int n_e, std::vector<int>* run_len) {
  Bounds b;
  b.b_sup = -INFINITY;
  b.mu_1 = INFINITY;
  b.norm_lower = 0.0;
  std::vector<std::pair<double, double>> nodes;  // (theta, weight)
  if (run_len) run_len->assign(nv, 0);
  for (int r = 0; r < nv; ++r) {
    // length of the run: stop at the first beta_j <= 1e-14 max|alpha_0..j|
    int len = steps;
    double amax = 0.0;
    for (int j = 0; j < steps; ++j) {
      amax = std::max(amax, std::fabs(alpha[(size_t)j * nv + r]));
      if (beta[(size_t)j * nv + r] <= 1e-14 * amax) {
        len = j + 1;
        break;
      }
    }
    if (run_len) (*run_len)[r] = len;
    std::vector<double> d(len), e(len);
    for (int j = 0; j < len; ++j) {
      d[j] = alpha[(size_t)j * nv + r];
      e[j] = beta[(size_t)j * nv + r];  // the last one is not part of the matrix
    }
    std::vector<double> th, y;
    tridiag_nodes(d, e, th, y);
    b.b_sup = std::max(b.b_sup, th[len - 1] + std::fabs(beta[(size_t)(len - 1) * nv + r]));
    b.mu_1 = std::min(b.mu_1, th[0]);
    b.norm_lower = std::max(b.norm_lower, std::max(std::fabs(th[0]), std::fabs(th[len - 1])));
    for (int j = 0; j < len; ++j) nodes.emplace_back(th[j], y[j] * y[j] / nv);
  }
  // density of states: smallest node where n * cumulative weight reaches n_e
  std::stable_sort(nodes.begin(), nodes.end(),
                   [](const std::pair<double, double>& x, const std::pair<double, double>& y) {
                     return x.first < y.first;
                   });
  const double target = (double)n_e - 1e-9 * (double)n_e;
  double cum = 0.0;
  b.mu_ne = nodes.back().first;
  for (auto& nw : nodes) {
    cum += nw.second;
    if (cum * (double)n >= target) {
      b.mu_ne = nw.first;
      break;
    }
  }
  b.mu_ne = std::min(std::max(b.mu_ne, b.mu_1), b.b_sup);
  return b;
}

std::vector<Coef> cheb_coefficients(int m, double b_sup, double mu_1, double mu_ne) {
  const double c = 0.5 * (b_sup + mu_ne), e = 0.5 * (b_sup - mu_ne);
  const double s1 = e / (mu_1 - c);
  std::vector<Coef> out;
  out.push_back({s1 / e, c, 0.0});
  double s = s1;
  for (int i = 2; i <= m; ++i) {
    const double sn = 1.0 / (2.0 / s1 - s);
    out.push_back({2.0 * sn / e, c, -s * sn});
    s = sn;
  }
  return out;
}

int optimal_degree(double res, double ritz, double c, double e, double tol, const chase_opts& o,
                   int deg) {
  int m;
  if (!o.optimize_degree) {
    m = deg;
  } else {
    const double t = (ritz - c) / e;
    double rho;
    if (std::fabs(t) <= 1.0) {
      rho = 1.0;  // |t +- i sqrt(1 - t^2)| = 1
    } else {
      const double r = std::sqrt(t * t - 1.0);
      rho = std::max(std::fabs(t + r), std::fabs(t - r));
    }
    if (rho <= 1.0 + 1e-12) {
      m = o.max_deg;
    } else {
      const double x = std::ceil(std::fabs(std::log(res / tol)) / std::log(rho));
      m = x > 1e6 ? o.max_deg : (int)x + o.deg_extra;
      m = std::min(m, o.max_deg);
    }
  }
  m = std::max(m, 2);
  m += m % 2;
  return m;
}

int fp64_tail_steps(double floor, double lam_nev, double c, double e, double tol, int deg) {
  if (!(e > 0.0) || !(floor > tol) || !(tol > 0.0)) return 0;
  const double t = (lam_nev - c) / e;
  if (!(t < -1.0)) return 0;
  const double rho = -t + std::sqrt(t * t - 1.0);
  const double j = std::ceil(std::log(floor / tol) / std::log(rho));
  return (std::isfinite(j) && j < deg) ? (int)j : 0;
}

double low_precision_floor(bool split_bf16, int64_t n) {
  if (split_bf16) return 0x1p-14;
  return 0x1p-17 * std::sqrt(std::max(1.0, (double)n / 3000.0));
}

}  // namespace chase
