// Host check of the Mueller screens (mueller.hpp): the regularisation of Eq. 6 and the refusal, before anything
// is allocated, of fields whose regularised matrix has a zero pivot at a lattice sample.  The device
// writes the screens, except at the samples that come within 1e-6 of singular or far from the normal range.
//
// A zero pivot of a singular matrix is a matter of rounding, so such a sample has one elimination that both decides
// and solves, `library::inverse`, in library complex arithmetic: another elimination may meet a zero where this
// one does not, and its screens would be NaN.  It costs ten times an elimination in plain arithmetic, which
// therefore goes first and leaves it those samples: 256^2 samples on 8 cores 28 ms with the library's
// arithmetic everywhere, 3.3 ms where no sample is close.
#include "mueller.hpp"

#include <algorithm>
#include <atomic>
#include <complex>
#include <mutex>
#include <thread>
#include <vector>

#include "common.hpp"

namespace pg {
namespace {

// Runs fn(begin, end) over [0, n) split across host threads (per-pixel work is independent).  fn throws nothing and
// allocates nothing: an exception in a thread ends the process.
template <class F>
void parallel_for(size_t n, F fn) {
  const size_t hw = std::max(1u, std::thread::hardware_concurrency());
  const size_t nt = std::min<size_t>({hw, 16, std::max<size_t>(1, n / 4096)});
  if (nt <= 1) {
    fn(size_t{0}, n);
    return;
  }
  std::vector<std::thread> th;
  const size_t step = (n + nt - 1) / nt;
  for (size_t t = 0; t < nt; ++t) {
    const size_t b = t * step, e = std::min(n, b + step);
    if (b < e) th.emplace_back(fn, b, e);
  }
  for (auto& x : th) x.join();
}

// Whether every pivot is far from zero: partial pivoting keeps the elimination's error below 1e-13 of the
// largest entry, so no order of the same elimination meets a zero.  NaN compares false.
bool far_from_singular(M4 m) {
  double top = 0.0;
  for (const auto& row : m.a)
    for (const cd& v : row) top = std::max(top, size_of(v));
  if (!(top > 1e-100 && top < 1e100)) return false;
  for (int col = 0; col < 4; ++col) {
    int piv = col;
    for (int r = col + 1; r < 4; ++r)
      if (size_of(m.a[r][col]) > size_of(m.a[piv][col])) piv = r;
    if (!(size_of(m.a[piv][col]) > 1e-6 * top)) return false;
    if (piv != col)
      for (int j = col; j < 4; ++j) std::swap(m.a[piv][j], m.a[col][j]);
    const cd inv = reciprocal(m.a[col][col]);
    for (int r = col + 1; r < 4; ++r) {
      const cd f = m.a[r][col] * inv;
      for (int j = col + 1; j < 4; ++j) m.a[r][j] = m.a[r][j] - f * m.a[col][j];
    }
  }
  return true;
}

namespace library {
using cd = std::complex<double>;
struct M4 {
  cd a[4][4];
};

M4 mul(const M4& x, const M4& y) {
  M4 r;
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j)
      for (int k = 0; k < 4; ++k) r.a[i][j] += x.a[i][k] * y.a[k][j];
  return r;
}

// S and S^-1 of Eq. 4; every entry is exact.
void stokes(int convention, M4& s, M4& sinv) {
  const cd u = convention == PG_STOKES_PAPER ? cd(0.0, 0.5) : cd(0.5, 0.0), i(0.0, 1.0);
  s = sinv = M4();
  s.a[0][0] = s.a[0][3] = s.a[1][0] = 0.5;
  s.a[1][3] = -0.5;
  s.a[2][1] = s.a[2][2] = u;
  s.a[3][1] = -0.5 * i;
  s.a[3][2] = 0.5 * i;
  sinv.a[0][0] = sinv.a[0][1] = sinv.a[3][0] = 1.0;
  sinv.a[3][1] = -1.0;
  sinv.a[1][2] = sinv.a[2][2] = 2.0 * std::conj(u);
  sinv.a[1][3] = i;
  sinv.a[2][3] = -i;
}

M4 mueller_at(const double* jones, const double* jones_b, size_t npix, size_t px, const M4& s, const M4& sinv) {
  cd ja[2][2], jb[2][2];
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      const size_t o = 2 * ((static_cast<size_t>(a) * 2 + b) * npix + px);
      ja[a][b] = jones ? cd(jones[o], jones[o + 1]) : cd(a == b ? 1.0 : 0.0);
      jb[a][b] = jones_b ? cd(jones_b[o], jones_b[o + 1]) : ja[a][b];
    }
  M4 m;
  for (int r = 0; r < 4; ++r)
    for (int c = 0; c < 4; ++c) m.a[r][c] = ja[r >> 1][c >> 1] * std::conj(jb[r & 1][c & 1]);
  return mul(mul(s, m), sinv);
}

// Gauss-Jordan with partial pivoting; false at a zero pivot.
bool inverse(const M4& m, M4& out) {
  cd w[4][8] = {};
  for (int i = 0; i < 4; ++i) {
    for (int j = 0; j < 4; ++j) w[i][j] = m.a[i][j];
    w[i][i + 4] = 1.0;
  }
  for (int col = 0; col < 4; ++col) {
    int piv = col;
    for (int r = col + 1; r < 4; ++r)
      if (std::abs(w[r][col]) > std::abs(w[piv][col])) piv = r;
    if (std::abs(w[piv][col]) == 0.0) return false;
    if (piv != col)
      for (int j = 0; j < 8; ++j) std::swap(w[piv][j], w[col][j]);
    const cd inv = 1.0 / w[col][col];
    for (int j = 0; j < 8; ++j) w[col][j] *= inv;
    for (int r = 0; r < 4; ++r) {
      if (r == col) continue;
      const cd f = w[r][col];
      if (f == 0.0) continue;
      for (int j = 0; j < 8; ++j) w[r][j] -= f * w[col][j];
    }
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) out.a[i][j] = w[i][j + 4];
  return true;
}
}  // namespace library

}  // namespace

bool check_screens(int npol, int kind, const double* jones, const double* jones_b, int mk, double eps, int convention,
                   ScreenCheck& out, std::string& err) {
  double(&beta)[4] = out.beta;
  for (double& b : beta) b = 0.0;
  out.px.clear();
  out.phi.clear();
  if (npol == 1 && (jones || jones_b)) {
    err = "npol = 1 (Stokes I only) takes no Jones field";
    return false;
  }
  if (npol == 1 || kind != PG_KIND_GRID) return true;
  const size_t npix = static_cast<size_t>(mk) * mk;
  const size_t samples = jones || jones_b ? npix : 1;  // no field: the same matrix everywhere
  const cd u = stokes_u(convention);
  std::mutex mu;
  parallel_for(samples, [&](size_t px0, size_t px1) {
    double mx[4] = {0.0, 0.0, 0.0, 0.0};
    for (size_t px = px0; px < px1; ++px) {
      const M4 m = mueller_at(jones, jones_b, npix, px, u);
      for (int p = 0; p < 4; ++p) mx[p] = std::max(mx[p], norm(m.a[p][p]));
    }
    std::lock_guard<std::mutex> lk(mu);
    for (int p = 0; p < 4; ++p) beta[p] = std::max(beta[p], mx[p]);
  });
  for (int p = 0; p < 4; ++p) beta[p] *= (eps / 2.0) * (eps / 2.0);
  std::vector<uint8_t> near(samples, 0);  // filled in by the threads, which allocate nothing: they have no one to throw to
  parallel_for(samples, [&](size_t px0, size_t px1) {
    for (size_t px = px0; px < px1; ++px) {
      M4 m = mueller_at(jones, jones_b, npix, px, u);
      regularise(m, beta);
      near[px] = !far_from_singular(m);
    }
  });
  std::vector<uint32_t>& close = out.px;
  close.reserve(std::count(near.begin(), near.end(), 1));
  for (size_t px = 0; px < samples; ++px)
    if (near[px]) close.push_back(static_cast<uint32_t>(px));
  if (samples == 1 && !close.empty()) {
    close.resize(npix);
    for (size_t px = 0; px < npix; ++px) close[px] = static_cast<uint32_t>(px);
  }
  std::atomic<bool> singular{false};
  if (!close.empty()) {
    out.phi.resize(32 * close.size());
    library::M4 s, sinv;
    library::stokes(convention, s, sinv);
    double top[4] = {0.0, 0.0, 0.0, 0.0};
    parallel_for(samples, [&](size_t px0, size_t px1) {
      double mx[4] = {0.0, 0.0, 0.0, 0.0};
      for (size_t px = px0; px < px1; ++px) {
        const library::M4 m = library::mueller_at(jones, jones_b, npix, px, s, sinv);
        for (int p = 0; p < 4; ++p) mx[p] = std::max(mx[p], std::abs(m.a[p][p]));
      }
      std::lock_guard<std::mutex> lk(mu);
      for (int p = 0; p < 4; ++p) top[p] = std::max(top[p], mx[p]);
    });
    parallel_for(close.size(), [&](size_t i0, size_t i1) {
      for (size_t i = i0; i < i1; ++i) {
        library::M4 m = library::mueller_at(jones, jones_b, npix, close[i], s, sinv);
        for (int p = 0; p < 4; ++p) {
          library::cd b = m.a[p][p];
          if (std::abs(b) == 0.0) b = 1e-150;
          const double weight = (eps / 2.0) * top[p] * (eps / 2.0) * top[p];
          m.a[p][p] = b * (1.0 + weight / std::norm(b));
        }
        library::M4 inv;
        if (!library::inverse(m, inv)) {
          singular = true;
          continue;
        }
        const library::M4 f = library::mul(inv, s);
        for (int qc = 0; qc < 16; ++qc) {
          out.phi[32 * i + 2 * qc] = f.a[qc / 4][qc % 4].real();
          out.phi[32 * i + 2 * qc + 1] = f.a[qc / 4][qc % 4].imag();
        }
      }
    });
  }
  if (singular) {
    err = "regularised Stokes Mueller matrix is singular at a lattice sample";
    return false;
  }
  return true;
}

}  // namespace pg
