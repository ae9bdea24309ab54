// Checks of the index arithmetic of the sums by distance bins
// (paper_2507_07823_amd/csrc/wfp_bins.h), built with UndefinedBehaviorSanitizer
// by tests/test_host_bins.py.  Exit status 0 when every check holds.
#include <cmath>
#include <cstdio>
#include <random>

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
// (1e30 apart), against the floor in floating point.
static void check_cells() {
  std::mt19937_64 g(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int k = 0; k < 400000; ++k) {
    const double dt = std::pow(10.0, -1.0 - 8.0 * u(g)), scale = 1500.0 * u(g) / dt + 1.0;
    const double e = u(g) < 0.3 ? 0.0 : 40.0 * dt * u(g);       // the chunk's lower edge
    const int c0 = (int)std::floor(e * scale) - 1, ctop = 1 + (int)(4094 * u(g));
    const double zs[] = {0.0, e, 50.0 * dt * u(g), 6.3 * u(g), 1e30, 2e30, (c0 + ctop) / scale, 2147483647.0 / scale};
    for (double z : zs) {
      const double want = std::fmax(std::fmin(std::floor(z * scale) - c0, ctop), 0.0);
      const int got = bin_cell(z, scale, c0, ctop);
      CHECK(got == (int)want, "cell of %.17g (scale %.17g, %d cells from %d): %d, not %d", z, scale, ctop + 1, c0, got,
            (int)want);
      if (failures > 5) return;
    }
  }
}

int main() {
  check_cells();
  if (failures) return 1;
  std::printf("bin checks passed\n");
  return 0;
}
