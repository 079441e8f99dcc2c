// Largest eigenvalue of a symmetric tridiagonal matrix and the last
// component of its eigenvector, and the basis change of a restart (host code;
// the Ritz steps of the Lanczos estimate of ||Theta_K||^2).
#pragma once

#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

namespace wdb {

// Largest eigenvalue of the symmetric tridiagonal matrix (diagonal a, off
// diagonal b) by bisection on the Sturm count, and the last component of its
// unit eigenvector by inverse iteration (tridiagonal elimination with
// partial pivoting).
struct TopRitz {
  double theta, last;
  std::vector<double> vec;  // the unit eigenvector (sign arbitrary)
};

inline int sturm_below(const std::vector<double>& a, const std::vector<double>& b, double x) {
  int cnt = 0;
  double q = 1.0;
  for (size_t i = 0; i < a.size(); ++i) {
    const double bb = i ? b[i - 1] * b[i - 1] : 0.0;
    q = a[i] - x - (i ? bb / q : 0.0);
    if (q == 0.0) q = -1e-300;
    if (q < 0.0) ++cnt;
  }
  return cnt;
}

inline TopRitz top_ritz(const std::vector<double>& a, const std::vector<double>& b) {
  const size_t m = a.size();
  double lo = a[0], hi = a[0];
  for (size_t i = 0; i < m; ++i) {
    const double r = (i ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(b[i]) : 0.0);
    lo = std::min(lo, a[i] - r);
    hi = std::max(hi, a[i] + r);
  }
  for (int it = 0; it < 200 && hi - lo > 0.0; ++it) {   // the top eigenvalue lies in (lo, hi]
    const double mid = 0.5 * (lo + hi);
    if (mid <= lo || mid >= hi) break;
    if (sturm_below(a, b, mid) == static_cast<int>(m)) hi = mid; else lo = mid;
  }
  const double theta = hi;
  if (m == 1) return TopRitz{theta, 1.0, std::vector<double>(1, 1.0)};
  // inverse iteration on (T - shift I), shift just above theta
  const double shift = theta + 4.0 * std::numeric_limits<double>::epsilon() * std::max(std::fabs(theta), 1e-300);
  std::vector<double> x(m, 1.0), dl(m), d(m), du(m), du2(m), rhs(m);
  for (int pass = 0; pass < 3; ++pass) {
    for (size_t i = 0; i < m; ++i) {
      d[i] = a[i] - shift;
      if (i + 1 < m) dl[i] = du[i] = b[i];
      du2[i] = 0.0;
      rhs[i] = x[i];
    }
    std::vector<int> piv(m, 0);
    for (size_t i = 0; i + 1 < m; ++i) {   // elimination with row interchanges
      if (std::fabs(d[i]) >= std::fabs(dl[i])) {
        const double f = d[i] != 0.0 ? dl[i] / d[i] : 0.0;
        d[i + 1] -= f * du[i];
        rhs[i + 1] -= f * rhs[i];
        if (i + 2 < m) du2[i] = 0.0;
      } else {
        const double f = d[i] / dl[i];
        d[i] = dl[i];
        const double t = d[i + 1];
        d[i + 1] = du[i] - f * t;
        du[i] = t;
        if (i + 2 < m) {
          du2[i] = du[i + 1];
          du[i + 1] = -f * du[i + 1];
        }
        std::swap(rhs[i], rhs[i + 1]);
        rhs[i + 1] -= f * rhs[i];
        piv[i] = 1;
      }
    }
    for (size_t k = m; k-- > 0;) {   // back substitution
      double t = rhs[k];
      if (k + 1 < m) t -= du[k] * x[k + 1];
      if (k + 2 < m) t -= du2[k] * x[k + 2];
      x[k] = d[k] != 0.0 ? t / d[k] : t / 1e-300;
    }
    double nrm = 0.0;
    for (double v : x) nrm += v * v;
    nrm = std::sqrt(nrm);
    for (double& v : x) v /= nrm;
  }
  return TopRitz{theta, x[m - 1], x};
}

// Eigenvalues (into a) and unit eigenvectors (rows of the result) of the symmetric
// tridiagonal matrix (a, b), by implicitly shifted QR steps with Wilkinson's shift
// (Golub and Van Loan, Matrix Computations, section 8.3).
inline std::vector<std::vector<double>> tridiag_eig(std::vector<double>& a, std::vector<double> b) {
  const int m = static_cast<int>(a.size());
  std::vector<std::vector<double>> S(m, std::vector<double>(m, 0.0));
  for (int i = 0; i < m; ++i) S[i][i] = 1.0;
  int hi = m - 1;
  for (int sweeps = 0; hi > 0 && sweeps < 60 * m; ++sweeps) {
    for (int i = 0; i < hi; ++i)
      if (std::fabs(b[i]) <= std::numeric_limits<double>::epsilon() * (std::fabs(a[i]) + std::fabs(a[i + 1]))) b[i] = 0.0;
    while (hi > 0 && b[hi - 1] == 0.0) --hi;
    if (hi == 0) break;
    int lo = hi - 1;
    while (lo > 0 && b[lo - 1] != 0.0) --lo;
    const double d = 0.5 * (a[hi - 1] - a[hi]), e = b[hi - 1];
    const double mu = a[hi] - e * e / (d + std::copysign(std::hypot(d, e), d));
    double x = a[lo] - mu, z = b[lo];
    for (int k = lo; k < hi; ++k) {   // rotate rows and columns k, k + 1 so that (x, z) becomes (r, 0)
      const double r = std::hypot(x, z);
      const double c = r > 0.0 ? x / r : 1.0, t = r > 0.0 ? z / r : 0.0;
      if (k > lo) b[k - 1] = r;
      const double ak = a[k], an = a[k + 1], bk = b[k];
      a[k] = c * c * ak + 2.0 * c * t * bk + t * t * an;
      a[k + 1] = t * t * ak - 2.0 * c * t * bk + c * c * an;
      b[k] = (c * c - t * t) * bk + c * t * (an - ak);
      if (k + 1 < hi) {
        x = b[k];
        z = t * b[k + 1];
        b[k + 1] *= c;
      }
      double *p = S[k].data(), *q = S[k + 1].data();
      for (int i = 0; i < m; ++i) {
        const double u = p[i], v = q[i];
        p[i] = c * u + t * v;
        q[i] = c * v - t * u;
      }
    }
  }
  return S;
}

// Restart of a Lanczos run M V = V T + bm v_m e_m^T (T of size m = a.size()): the
// columns of C (m x l, row major) combine V to l vectors that span the Ritz vectors
// of the l largest Ritz values, in which M stays tridiagonal: V C, v_m is the
// start of a run with the diagonal a (l entries) and off-diagonal b (l entries,
// the last couples v_m).
struct Restart {
  std::vector<double> C, a, b;
};

inline Restart restart_basis(std::vector<double> a, const std::vector<double>& b, double bm, int l) {
  const int m = static_cast<int>(a.size());
  const auto S = tridiag_eig(a, b);
  std::vector<int> order(m);
  for (int i = 0; i < m; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int i, int j) { return a[i] > a[j]; });
  // In the Ritz vectors M is diagonal with the row bm S_i[m - 1] below.  Householder
  // reflections from that row upwards make it tridiagonal (Q on the Ritz vectors).
  const int n = l + 1;
  std::vector<double> A(static_cast<size_t>(n) * n, 0.0), Q(static_cast<size_t>(l) * l, 0.0);
  for (int i = 0; i < l; ++i) {
    A[static_cast<size_t>(i) * n + i] = a[order[i]];
    A[static_cast<size_t>(l) * n + i] = A[static_cast<size_t>(i) * n + l] = bm * S[order[i]][m - 1];
    Q[static_cast<size_t>(i) * l + i] = 1.0;
  }
  for (int row = l; row >= 2; --row) {   // entries 0 .. row - 2 of this row vanish
    std::vector<double> h(A.begin() + static_cast<size_t>(row) * n, A.begin() + static_cast<size_t>(row) * n + row);
    double nrm = 0.0, off = 0.0;
    for (int i = 0; i < row; ++i) nrm += h[i] * h[i];
    for (int i = 0; i + 1 < row; ++i) off += h[i] * h[i];
    if (off == 0.0) continue;
    h[row - 1] += std::copysign(std::sqrt(nrm), h[row - 1]);
    const double hh = off + h[row - 1] * h[row - 1];
    const auto reflect = [&](std::vector<double>& X, int rows, int cols, int ld, bool left) {   // X -= 2/hh (h h^T) X
      for (int j = 0; j < (left ? cols : rows); ++j) {
        const auto at = [&](int i) -> double& { return left ? X[static_cast<size_t>(i) * ld + j] : X[static_cast<size_t>(j) * ld + i]; };
        double t = 0.0;
        for (int i = 0; i < row; ++i) t += h[i] * at(i);
        t *= 2.0 / hh;
        for (int i = 0; i < row; ++i) at(i) -= t * h[i];
      }
    };
    reflect(A, n, n, n, true);
    reflect(A, n, n, n, false);
    reflect(Q, l, l, l, false);
  }
  Restart r;
  r.C.assign(static_cast<size_t>(m) * l, 0.0);
  for (int i = 0; i < m; ++i)
    for (int k = 0; k < l; ++k) {
      const double v = S[order[k]][i];
      for (int j = 0; j < l; ++j) r.C[static_cast<size_t>(i) * l + j] += v * Q[static_cast<size_t>(k) * l + j];
    }
  for (int i = 0; i < l; ++i) {
    r.a.push_back(A[static_cast<size_t>(i) * n + i]);
    r.b.push_back(A[static_cast<size_t>(i + 1) * n + i]);
  }
  return r;
}

}  // namespace wdb
