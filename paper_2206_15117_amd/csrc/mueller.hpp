// Image-domain screens Phi_qc(l, m) of the Mueller kernels at one lattice sample, float64, for the device
// (which writes the screens) and the host's check of the field.
//
// Sec. 3.2: Mueller matrices from the Jones matrices of a baseline's two antennas,
// M = J_a (x) conj(J_b) (identical antennas: J_b = J_a) in correlation order XX, XY, YX, YY (Eq. 3); Stokes form
// M^S = S M S^-1 with S from Eq. 4 (U = (XY + YX)/2 by default, the printed
// U = i (XY + YX)/2 on request).  Gridding screens are (M'^S)^-1 S, where M' has
// its diagonal regularised by Eq. 6 (Sec. 3.3); degridding screens are
// (S^-1 M^S)^H, whose conjugate carries the Stokes sky to observed correlations.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>

#include "polgrid.h"

// No product is fused into a sum here: host and device see the same matrices.
#pragma clang fp contract(off)

namespace pg {

// Written out: std::complex products and quotients test for infinities.
struct cd {
  double re, im;
};
__host__ __device__ inline cd operator+(cd x, cd y) { return {x.re + y.re, x.im + y.im}; }
__host__ __device__ inline cd operator-(cd x, cd y) { return {x.re - y.re, x.im - y.im}; }
__host__ __device__ inline cd operator*(cd x, cd y) { return {x.re * y.re - x.im * y.im, x.re * y.im + x.im * y.re}; }
__host__ __device__ inline cd operator*(double f, cd x) { return {f * x.re, f * x.im}; }
__host__ __device__ inline cd conj(cd x) { return {x.re, -x.im}; }
__host__ __device__ inline double norm(cd x) { return x.re * x.re + x.im * x.im; }
// 1-norm: zero exactly where x is, finite where the squared magnitude is not
__host__ __device__ inline double size_of(cd x) { return fabs(x.re) + fabs(x.im); }
__host__ __device__ inline cd reciprocal(cd x) {
  const double m = size_of(x);
  const cd y{x.re / m, x.im / m};
  const double d = 1.0 / (norm(y) * m);
  return {y.re * d, -y.im * d};
}

struct M4 {
  cd a[4][4];
};

// S of Eq. 4: I and Q from (XX, YY), U and V from (XY, YX); u is 1/2 or, as printed, i/2.
__host__ __device__ inline cd stokes_u(int convention) {
  return convention == PG_STOKES_PAPER ? cd{0.0, 0.5} : cd{0.5, 0.0};
}
__host__ __device__ inline M4 stokes(int convention) {
  M4 s = {};
  const cd u = stokes_u(convention);
  s.a[0][0] = s.a[0][3] = s.a[1][0] = {0.5, 0.0};
  s.a[1][3] = {-0.5, 0.0};
  s.a[2][1] = s.a[2][2] = u;
  s.a[3][1] = {0.0, -0.5};
  s.a[3][2] = {0.0, 0.5};
  return s;
}

// S x and S^-1 x for a column x (XX, XY, YX, YY), x S^-1 for a row: two terms to an entry.
// S^-1: XX = I + Q, YY = I - Q, XY = U / (2 u) + i V, YX = U / (2 u) - i V.
__host__ __device__ inline void stokes_times(cd u, const cd x[4], cd y[4]) {
  const cd d = x[2] - x[1];
  y[0] = 0.5 * (x[0] + x[3]);
  y[1] = 0.5 * (x[0] - x[3]);
  y[2] = u * (x[1] + x[2]);
  y[3] = {-0.5 * d.im, 0.5 * d.re};
}
__host__ __device__ inline void stokes_inverse_times(cd u, const cd x[4], cd y[4]) {
  const cd t = cd{2.0 * u.re, -2.0 * u.im} * x[2];  // 1 / (2 u) = 2 conj(u)
  const cd iv = {-x[3].im, x[3].re};
  y[0] = x[0] + x[1];
  y[3] = x[0] - x[1];
  y[1] = t + iv;
  y[2] = t - iv;
}
__host__ __device__ inline void times_stokes_inverse(cd u, const cd x[4], cd y[4]) {
  const cd d = x[1] - x[2];
  y[0] = x[0] + x[3];
  y[1] = x[0] - x[3];
  y[2] = cd{2.0 * u.re, -2.0 * u.im} * (x[1] + x[2]);
  y[3] = {-d.im, d.re};
}

// M^S at sample px of the lattice: J_a from `jones`, J_b from `jones_b` (identical antennas when NULL;
// the identity when both are).  Fields are [2][2][npix], (re, im).
__host__ __device__ inline M4 mueller_at(const double* jones, const double* jones_b, size_t npix, size_t px, cd u) {
  cd ja[2][2], jb[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const size_t o = 2 * ((static_cast<size_t>(a) * 2 + b) * npix + px);
      ja[a][b] = jones ? cd{jones[o], jones[o + 1]} : cd{a == b ? 1.0 : 0.0, 0.0};
      jb[a][b] = jones_b ? cd{jones_b[o], jones_b[o + 1]} : ja[a][b];
    }
  M4 m;
#pragma unroll
  for (int c = 0; c < 4; ++c) {  // column (c, d) of J_a (x) conj(J_b), then S from the left
    cd col[4], y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) col[r] = ja[r >> 1][c >> 1] * conj(jb[r & 1][c & 1]);
    stokes_times(u, col, y);
#pragma unroll
    for (int r = 0; r < 4; ++r) m.a[r][c] = y[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    cd y[4];
    times_stokes_inverse(u, m.a[r], y);
#pragma unroll
    for (int c = 0; c < 4; ++c) m.a[r][c] = y[c];
  }
  return m;
}

// Eq. 6 on the diagonal, beta[p] = (eps / 2 max |M^S_pp|)^2.
__host__ __device__ inline void regularise(M4& m, const double beta[4]) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    cd b = m.a[p][p];
    if (size_of(b) == 0.0) b = {1e-150, 0.0};
    m.a[p][p] = (1.0 + beta[p] / norm(b)) * b;
  }
}

// x <- m^-1 x, m overwritten, by Gauss-Jordan elimination with partial pivoting.  Rows move by selects:
// registers have no address.
__host__ __device__ inline void solve(M4& m, M4& x) {
#pragma unroll
  for (int col = 0; col < 4; ++col) {
#pragma unroll
    for (int r = col + 1; r < 4; ++r)
      if (size_of(m.a[r][col]) > size_of(m.a[col][col])) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const cd t = m.a[r][j], v = x.a[r][j];
          m.a[r][j] = m.a[col][j];
          x.a[r][j] = x.a[col][j];
          m.a[col][j] = t;
          x.a[col][j] = v;
        }
      }
    const cd inv = reciprocal(m.a[col][col]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j > col) m.a[col][j] = inv * m.a[col][j];
      x.a[col][j] = inv * x.a[col][j];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r == col) continue;
      const cd f = m.a[r][col];
      if (size_of(f) == 0.0) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j > col) m.a[r][j] = m.a[r][j] - f * m.a[col][j];
        x.a[r][j] = x.a[r][j] - f * x.a[col][j];
      }
    }
  }
}

}  // namespace pg

#pragma clang fp contract(fast)  // what HIP code is compiled with otherwise
