// Host check of the Mueller screens (mueller.hpp): the regularisation of Eq. 6 and the refusal of fields
// whose regularised matrix is singular at a lattice sample.  The device writes the screens.
#include "mueller.hpp"

#include <algorithm>
#include <atomic>
#include <mutex>
#include <thread>
#include <vector>

#include "common.hpp"

namespace pg {
namespace {

// Runs fn(begin, end) over [0, n) split across host threads (per-pixel work is independent).
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

}  // namespace

bool check_screens(int npol, int kind, const double* jones, const double* jones_b, int mk, double eps, int convention,
                   double beta[4], std::string& err) {
  for (int p = 0; p < 4; ++p) beta[p] = 0.0;
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
  std::atomic<bool> singular{false};
  parallel_for(samples, [&](size_t px0, size_t px1) {
    for (size_t px = px0; px < px1; ++px) {
      M4 m = mueller_at(jones, jones_b, npix, px, u);
      regularise(m, beta);
      if (!solve(m, nullptr)) singular = true;
    }
  });
  if (singular) {
    err = "regularised Stokes Mueller matrix is singular at a lattice sample";
    return false;
  }
  return true;
}

}  // namespace pg
