// The host's check of Mueller screens against what the device does with its result, on the CPU: every sample of an
// accepted finite field has finite screens, the check's own where it lists the sample, otherwise those of
// the elimination that the device runs.  With the argument `threads`: a field of singular samples large enough to be
// split over threads, while every allocation outside the main thread fails.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "common.hpp"
#include "mueller.hpp"

namespace {
const std::thread::id g_main = std::this_thread::get_id();
bool g_main_only = false;
}  // namespace

void* operator new(std::size_t n) {
  if (g_main_only && std::this_thread::get_id() != g_main) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

namespace {

struct Tally {
  int accepted = 0, refused = 0, listed = 0, not_finite = 0;
};

bool finite(const pg::M4& f) {
  for (const auto& row : f.a)
    for (const pg::cd& v : row)
      if (!std::isfinite(v.re) || !std::isfinite(v.im)) return false;
  return true;
}

void check(const std::vector<double>& ja, const std::vector<double>& jb, int mk, double eps, int convention, Tally& t) {
  const size_t npix = static_cast<size_t>(mk) * mk;
  const double *a = ja.empty() ? nullptr : ja.data(), *b = jb.empty() ? nullptr : jb.data();
  pg::ScreenCheck out;
  std::string err;
  if (!pg::check_screens(4, PG_KIND_GRID, a, b, mk, eps, convention, out, err)) {
    ++t.refused;
    return;
  }
  ++t.accepted;
  std::vector<char> listed(npix, 0);
  for (size_t i = 0; i < out.px.size(); ++i) {
    listed[out.px[i]] = 1;
    ++t.listed;
    for (int e = 0; e < 32; ++e)
      if (!std::isfinite(out.phi[32 * i + e])) {
        ++t.not_finite;
        break;
      }
  }
  for (size_t px = 0; px < npix; ++px) {
    if (listed[px]) continue;
    pg::M4 m = pg::mueller_at(a, b, npix, px, pg::stokes_u(convention)), f = pg::stokes(convention);
    pg::regularise(m, out.beta);
    pg::solve(m, f);
    if (!finite(f)) ++t.not_finite;
  }
}

int threads() {
  const int mk = 128;
  std::vector<double> field(8 * mk * mk, 0.0);
  for (size_t i = 0; i < field.size(); i += 2) field[i] = i < 4u * mk * mk ? 0.3 : 0.7;
  pg::ScreenCheck out;
  std::string err;
  g_main_only = true;
  const bool refused = !pg::check_screens(4, PG_KIND_GRID, field.data(), nullptr, mk, 0.0, PG_STOKES_IAU, out, err);
  g_main_only = false;
  std::printf("%s, %zu samples near\n", refused ? "refused" : "accepted", out.px.size());
  return out.px.size() == static_cast<size_t>(mk) * mk ? 0 : 1;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc > 1 && std::string(argv[1]) == "threads") return threads();
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  Tally t;
  const int mk = 4, npix = mk * mk;
  // rows (a, b) and f (a, b), values in tenths: rank one, with and without an imaginary part
  for (int n = 0; n < 4000; ++n) {
    const bool complex_field = n % 2, two = n % 4 > 1;
    std::vector<double> field[2];
    for (int k = 0; k <= (two ? 1 : 0); ++k) {
      field[k].assign(8 * npix, 0.0);
      for (int px = 0; px < npix; ++px) {
        double row[2][2], f[2];
        const auto tenth = [&] { return std::round(10.0 * u(rng)) / 10.0; };
        for (auto& v : row)
          for (double& x : v) x = tenth();
        for (double& x : f) x = tenth();
        if (!complex_field) row[0][1] = row[1][1] = f[1] = 0.0;
        for (int c = 0; c < 2; ++c) {
          const double re = row[c][0], im = row[c][1];
          field[k][2 * (c * npix + px)] = re;
          field[k][2 * (c * npix + px) + 1] = im;
          field[k][2 * ((2 + c) * npix + px)] = re * f[0] - im * f[1];
          field[k][2 * ((2 + c) * npix + px) + 1] = re * f[1] + im * f[0];
        }
      }
    }
    // most such fields meet a zero at one of their samples: the same sample everywhere tells them apart
    for (auto& j : field)
      for (size_t e = 0; e + 1 < j.size(); e += 2)
        for (int i = 0; i < 2; ++i) j[e + i] = j[2 * (e / 2 / npix * npix) + i];
    check(field[0], field[1], mk, n % 8 > 5 ? 0.2 : 0.0, n % 3 ? PG_STOKES_IAU : PG_STOKES_PAPER, t);
  }
  check({}, {}, mk, 0.2, PG_STOKES_IAU, t);
  std::printf("accepted %d refused %d listed %d not finite %d\n", t.accepted, t.refused, t.listed, t.not_finite);
  return t.not_finite == 0 && t.accepted > 500 && t.refused > 100 && t.listed > 1000 ? 0 : 1;
}
