// Checks of the index arithmetic of the sums by distance bins
// (paper_2507_07823_amd/csrc/wfp_bins.h), built with UndefinedBehaviorSanitizer
// by tests/test_host_bins.py.  Exit status 0 when every check holds.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2507_07823_amd/csrc/wfp_bins.h"

using namespace wfp;

static int failures = 0;
#define CHECK(c, ...)                                           \
  do {                                                          \
    if (!(c)) {                                                 \
      std::fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
      std::fprintf(stderr, __VA_ARGS__);                        \
      std::fprintf(stderr, "\n");                               \
      ++failures;                                               \
    }                                                           \
  } while (0)

// Any distance, across the box and the stand-ins of missing sources and targets
// (1e30 apart, or 2 pi less that), against the floor in floating point.
static void check_cells() {
  std::mt19937_64 g(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int k = 0; k < 400000; ++k) {
    const double dt = std::pow(10.0, -1.0 - 8.0 * u(g)), scale = 1500.0 * u(g) / dt + 1.0;
    const double e = u(g) < 0.3 ? 0.0 : 40.0 * dt * u(g);       // the chunk's lower edge
    const int c0 = (int)std::floor(e * scale) - 1, ctop = 1 + (int)(4094 * u(g));
    const double zs[] = {0.0, e, 50.0 * dt * u(g), 6.3 * u(g), 1e30, 2e30, 6.3 - 1e30, -6.3 * u(g), (c0 + ctop) / scale, 2147483647.0 / scale};
    for (double z : zs) {
      const double want = std::fmax(std::fmin(std::floor(std::fabs(z) * scale) - c0, ctop), 0.0);
      const int got = bin_cell(z, scale, c0, ctop);
      CHECK(got == (int)want, "cell of %.17g (scale %.17g, %d cells from %d): %d, not %d", z, scale, ctop + 1, c0, got,
            (int)want);
      if (failures > 5) return;
    }
  }
}

// Every pair whose distance, as the sum computes it, lies in a chunk has its
// target in the chunk's window: springs at the chunk's edges from one another, to
// the last places, at steps down to 1e-7 (where the rounding of the coordinates
// outweighs any fixed part of the step).
static void check_windows() {
  constexpr double pi = 3.14159265358979323846;
  std::mt19937_64 g(9);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int k = 0; k < 3000; ++k) {
    const double dt = std::pow(10.0, -2.0 - 5.0 * u(g)), elo = 30.0 * dt * u(g), ehi = elo + 3.0 * dt;
    const bool periodic = k % 2, seam = periodic && k % 4 == 1;
    std::vector<double> xs;
    const double base = seam ? pi - 20.0 * dt * u(g) : 6.0 * (u(g) - 0.5);
    auto add = [&](double x) {
      if (x >= pi) x -= 2.0 * pi;
      if (periodic || std::fabs(x) < pi) xs.push_back(x);
    };
    for (int i = 0; i < 6; ++i) {
      const double x = base + dt * u(g);
      add(x);
      for (double e : {elo, ehi})
        for (int n = -3; n <= 3; ++n)
          for (int side : {-1, 1}) add(x + side * e + n * 2.2e-16);
    }
    std::sort(xs.begin(), xs.end());
    const int M = (int)xs.size(), nsrc = 8;
    for (int b = 0; b * nsrc < M; ++b) {
      const int j1 = std::min((b + 1) * nsrc, M);
      const BinWindow w = bin_window(xs.data(), M, periodic, xs[b * nsrc], xs[j1 - 1], elo, ehi, bin_tol(dt), false);
      CHECK(w.l0 <= w.l1 && w.r0 <= w.r1 && (w.l1 <= w.r0 || w.l1 == w.l0), "overlapping runs");
      for (int j = b * nsrc; j < j1; ++j)
        for (int v = periodic ? -M : 0; v < (periodic ? 2 * M : M); ++v) {
          const double x = xs[v < 0 ? v + M : (v >= M ? v - M : v)];
          double z = std::fabs(x - xs[j]);
          if (v < 0 || v >= M) {
            if (v < 0 ? x < xs[j] : x > xs[j]) continue;      // more than a turn apart
            z = 2.0 * pi - z;
          }
          if (!(z >= elo && z < ehi)) continue;
          CHECK((v >= w.l0 && v < w.l1) || (v >= w.r0 && v < w.r1), "target %d of source %d (%.17g in [%.17g, %.17g), dt %g)",
                v, j, z, elo, ehi, dt);
          if (failures > 5) return;
        }
    }
  }
}

int main() {
  check_cells();
  check_windows();
  if (failures) return 1;
  std::printf("bin checks passed\n");
  return 0;
}
