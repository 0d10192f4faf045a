// Order-0 prolate spheroidal wave function psi_0(c, x) on [-1, 1], float64.
//
// The anti-aliasing function multiplied into every kernel in the image domain
// (Sec. 3.2).  Method: expand psi_0 in even normalised Legendre polynomials;
// the coefficient vector is the eigenvector of the smallest eigenvalue of the
// (symmetric, tridiagonal) matrix of the prolate differential operator
//   -d/dx (1 - x^2) d/dx + c^2 x^2
// in that basis (Bouwkamp 1947; Xiao, Rokhlin & Yarvin 2001).  The matrix is positive definite and its
// eigenvalues lie about c (2k + 1), k = 0, 2, 4, ... apart, so inverse iteration gains a factor of five
// a step; 48 steps are far past rounding.  (Jacobi rotations of the dense matrix took milliseconds.)
#include <cmath>
#include <vector>

#include "common.hpp"

namespace pg {
namespace {

// Eigenvector of the smallest eigenvalue of the positive definite tridiagonal matrix with diagonal d
// and off-diagonal e, by inverse iteration on its L D L^T factors.
std::vector<double> smallest_eigenvector(std::vector<double> d, const std::vector<double>& e) {
  const int n = static_cast<int>(d.size());
  std::vector<double> l(n, 0.0), v(n, 0.0);
  for (int i = 1; i < n; ++i) {
    l[i] = e[i - 1] / d[i - 1];
    d[i] -= l[i] * e[i - 1];
  }
  v[0] = 1.0;
  for (int it = 0; it < 48; ++it) {
    for (int i = 1; i < n; ++i) v[i] -= l[i] * v[i - 1];
    for (int i = 0; i < n; ++i) v[i] /= d[i];
    for (int i = n - 2; i >= 0; --i) v[i] -= l[i + 1] * v[i + 1];
    double s = 0.0;
    for (double x : v) s += x * x;
    s = 1.0 / std::sqrt(s);
    for (double& x : v) x *= s;
  }
  return v;
}

// sum_i coef[i] P_{2i}(x) at every x, by the Legendre three-term recurrence (points in the inner loop:
// they are independent, the degrees are a chain).
std::vector<double> even_legendre_series(const std::vector<double>& coef, const std::vector<double>& x) {
  const size_t m = x.size();
  std::vector<double> p0(m, 1.0), p1(x), sum(m, coef[0]);
  const int deg_max = 2 * (static_cast<int>(coef.size()) - 1);
  for (int k = 1; k < deg_max; ++k) {
    const double a = (2.0 * k + 1.0) / (k + 1), b = static_cast<double>(k) / (k + 1);
    const double c = (k + 1) % 2 == 0 ? coef[(k + 1) / 2] : 0.0;
    for (size_t i = 0; i < m; ++i) {
      const double p2 = a * x[i] * p1[i] - b * p0[i];
      p0[i] = p1[i];
      p1[i] = p2;
      sum[i] += c * p2;
    }
  }
  return sum;
}

}  // namespace

std::vector<double> pswf0(double c, const std::vector<double>& x) {
  const int n = static_cast<int>(c) + 40;
  std::vector<double> d(n), e(n - 1);
  for (int i = 0; i < n; ++i) {
    const double k = 2.0 * i;
    d[i] = k * (k + 1) + c * c * (2 * k * (k + 1) - 1) / ((2 * k + 3) * (2 * k - 1));
    if (i + 1 < n) e[i] = c * c * (k + 2) * (k + 1) / ((2 * k + 3) * std::sqrt((2 * k + 1) * (2 * k + 5)));
  }
  std::vector<double> coef = smallest_eigenvector(d, e);
  for (int i = 0; i < n; ++i) coef[i] *= std::sqrt(2.0 * i + 0.5);  // normalised -> plain basis
  std::vector<double> out = even_legendre_series(coef, x);
  const double norm = even_legendre_series(coef, {0.0})[0];
  for (double& v : out) v /= norm;
  return out;
}

}  // namespace pg
