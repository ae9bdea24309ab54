// Checks of the local sum's forms (paper_2507_07823_amd/csrc/wfp_forms.cpp), built
// with the sanitizers by tests/test_host_bins.py: the look-up of a distance's bin
// over the layouts, and the rules against measured times.  Exit status 0 when
// every check holds.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2507_07823_amd/csrc/wfp_bins.h"
#include "../../paper_2507_07823_amd/csrc/wfp_forms.h"
#include "../../paper_2507_07823_amd/csrc/wfp_host.h"

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

static bool layout(int W, int p, double eps, int ngl, double dt, BinLayout& B) {
  std::vector<double> z, w;
  gauss_legendre(ngl, z, w);
  return bin_layout(W, p, std::log(1.0 / eps), dt, z, B);
}

// The kernel's look-up of a distance in a chunk: the cell's record, then at most
// `bumps` edges (two for the kernel of layouts with one), record r = bin r - 1.
static int look_up(const BinLayout& B, int c, double z) {
  const int* ch = B.chunk[c].data();
  const int at = bin_cell(z, B.scales[c], ch[0], ch[1] - 1);
  CHECK(at >= 0 && at < ch[1] && 4 * ch[2] + at < (int)B.cells.size(), "cell %d of %d", at, ch[1]);
  int r = B.cells[4 * ch[2] + at];
  const int bumps = B.ks == 13 ? 4 : std::max(1, B.bumps);
  for (int s = 0; s < bumps; ++s) {
    const double top = r <= kBinChunk ? B.edge[c * kBinChunk + r] : 1e300;
    if (z >= top) ++r;
  }
  return r;
}

static void check_look_up() {
  std::mt19937_64 g(3);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  int fits = 0;
  for (int p : {2, 4, 6, 8})
    for (double eps : {1e-3, 1e-6, 1e-9, 1e-12})
      for (double dt : {5e-3, 1e-5, 2e-7}) {
        const int W = (int)std::lround(2.0 * std::log(1.0 / eps) / (kPi * 0.5));
        for (int ngl : {W, 30}) {
          BinLayout B;
          if (!layout(W, p, eps, ngl, dt, B)) continue;
          ++fits;
          CHECK(B.bumps >= 1 && B.bumps <= 4 && (B.ks == 13 || (B.bumps <= 2 && W + p / 2 <= 40)), "kernel limits");
          std::vector<double> zs{0.0, W * dt, 1.0, 6.0, 1e30};
          for (int i = 0; i < 2000; ++i) zs.push_back(1.1 * W * dt * u(g));
          for (double e : B.edge)
            for (int k = -1; k <= 1; ++k) zs.push_back(std::fabs(e * (1.0 + k * 2.3e-16)));
          for (double z : zs)
            for (int c = 0; c < B.nch; ++c) {
              const int r = look_up(B, c, z);
              const double* e = &B.edge[c * kBinChunk];
              // below the chunk, in its bin r - 1, or above (empty bins and beyond)
              const bool ok = z < e[0] ? r == 0 : (z >= e[kBinChunk] ? r >= 1 && (r == kBinChunk + 1 || e[r - 1] == e[r])
                                                                      : r >= 1 && r <= kBinChunk && z >= e[r - 1] && z < e[r]);
              CHECK(ok, "W %d p %d eps %g: distance %.17g in chunk %d: record %d", W, p, eps, z, c, r);
              if (failures > 5) return;
            }
        }
      }
  CHECK(fits >= 60, "%d layouts fit", fits);
  // limits: too many bins, too high an order
  BinLayout B;
  CHECK(!layout(4, 8, 5e-3, 4, 1e-3, B) && !layout(1, 2, 0.3, 1, 1e-3, B) && layout(5, 8, 5e-3, 5, 1e-3, B),
        "windows too short for the stencil");
  CHECK(!layout(37, 8, 1e-12, 37, 1e-3, B) && !layout(35, 8, 1e-12, 40, 1e-3, B) && !layout(35, 10, 1e-12, 35, 1e-3, B),
        "layouts beyond the limits");
  CHECK(layout(18, 8, 1e-6, 18, 1e-3, B) && B.ks == 13 && layout(36, 8, 1e-12, 36, 1e-3, B) && B.ks == 10, "steps");
}

// Measured levels: time pair by pair over time by bins, at so many springs and
// neighbours, of marches and gradients.  The rule takes no form that measured
// 1.1 times slower, nor leaves one that measured 1.3 times faster.
struct Row {
  int W;
  double eps;
  int p, M, n, gradient;
  double ratio;
};
static const Row kRows[] = {
    {35, 1e-12, 8, 3000, 159, 0, 0.90}, {35, 1e-12, 8, 2000, 174, 0, 0.85},
    {35, 1e-12, 2, 2000, 134, 0, 0.589}, {35, 1e-12, 2, 2000, 223, 0, 0.697}, {35, 1e-12, 2, 2000, 379, 0, 0.841},
    {35, 1e-12, 2, 20000, 137, 0, 0.681}, {35, 1e-12, 2, 20000, 231, 0, 0.833},
    {35, 1e-12, 2, 20000, 398, 0, 1.059}, {35, 1e-12, 2, 100000, 137, 0, 0.660},
    {35, 1e-12, 2, 100000, 231, 0, 0.757}, {35, 1e-12, 2, 100000, 400, 0, 1.113},
    {35, 1e-12, 4, 2000, 134, 0, 0.674}, {35, 1e-12, 4, 2000, 223, 0, 0.799}, {35, 1e-12, 4, 2000, 379, 0, 0.968},
    {35, 1e-12, 4, 20000, 137, 0, 0.833}, {35, 1e-12, 4, 20000, 231, 0, 1.015},
    {35, 1e-12, 4, 20000, 398, 0, 1.369}, {35, 1e-12, 4, 100000, 137, 0, 0.829},
    {35, 1e-12, 4, 100000, 231, 0, 0.960}, {35, 1e-12, 4, 100000, 400, 0, 1.449},
    {35, 1e-12, 6, 2000, 134, 0, 0.809}, {35, 1e-12, 6, 2000, 223, 0, 0.937}, {35, 1e-12, 6, 2000, 379, 0, 1.162},
    {35, 1e-12, 6, 20000, 137, 0, 1.023}, {35, 1e-12, 6, 20000, 231, 0, 1.239},
    {35, 1e-12, 6, 20000, 398, 0, 1.640}, {35, 1e-12, 6, 100000, 137, 0, 1.047},
    {35, 1e-12, 6, 100000, 231, 0, 1.220}, {35, 1e-12, 6, 100000, 400, 0, 1.858},
    {35, 1e-12, 8, 2000, 134, 0, 0.917}, {35, 1e-12, 8, 2000, 223, 0, 1.056}, {35, 1e-12, 8, 2000, 379, 0, 1.312},
    {35, 1e-12, 8, 20000, 137, 0, 1.201}, {35, 1e-12, 8, 20000, 231, 0, 1.449},
    {35, 1e-12, 8, 20000, 398, 0, 1.974}, {35, 1e-12, 8, 100000, 137, 0, 1.246},
    {35, 1e-12, 8, 100000, 231, 0, 1.455}, {35, 1e-12, 8, 100000, 400, 0, 2.244},
    {18, 1e-06, 2, 2000, 134, 0, 0.771}, {18, 1e-06, 2, 2000, 379, 0, 0.969},
    {18, 1e-06, 2, 20000, 137, 0, 0.819}, {18, 1e-06, 2, 20000, 231, 0, 0.937},
    {18, 1e-06, 2, 20000, 398, 0, 1.149}, {18, 1e-06, 4, 2000, 134, 0, 0.751},
    {18, 1e-06, 4, 2000, 379, 0, 0.946}, {18, 1e-06, 4, 20000, 137, 0, 0.816},
    {18, 1e-06, 4, 20000, 231, 0, 0.956}, {18, 1e-06, 4, 20000, 398, 0, 1.194},
    {18, 1e-06, 6, 2000, 134, 0, 0.819}, {18, 1e-06, 6, 2000, 379, 0, 1.044},
    {18, 1e-06, 6, 20000, 137, 0, 0.914}, {18, 1e-06, 6, 20000, 231, 0, 1.065},
    {18, 1e-06, 6, 20000, 398, 0, 1.349}, {18, 1e-06, 8, 2000, 134, 0, 0.951},
    {18, 1e-06, 8, 2000, 379, 0, 1.214}, {18, 1e-06, 8, 20000, 137, 0, 1.153},
    {18, 1e-06, 8, 20000, 231, 0, 1.344}, {18, 1e-06, 8, 20000, 398, 0, 1.732},
    {20, 1e-12, 2, 20000, 137, 0, 0.653}, {20, 1e-12, 2, 20000, 231, 0, 0.756},
    {20, 1e-12, 2, 20000, 398, 0, 0.952}, {20, 1e-12, 4, 20000, 137, 0, 0.745},
    {20, 1e-12, 4, 20000, 231, 0, 0.883}, {20, 1e-12, 4, 20000, 398, 0, 1.128},
    {20, 1e-12, 6, 20000, 137, 0, 0.848}, {20, 1e-12, 6, 20000, 231, 0, 1.014},
    {20, 1e-12, 6, 20000, 398, 0, 1.325}, {20, 1e-12, 8, 20000, 137, 0, 1.024},
    {20, 1e-12, 8, 20000, 231, 0, 1.239}, {20, 1e-12, 8, 20000, 398, 0, 1.653},
    {35, 1e-12, 2, 30000, 137, 1, 0.527}, {35, 1e-12, 2, 30000, 231, 1, 0.762},
    {35, 1e-12, 2, 30000, 399, 1, 1.027}, {35, 1e-12, 4, 30000, 137, 1, 0.648},
    {35, 1e-12, 4, 30000, 231, 1, 0.948}, {35, 1e-12, 4, 30000, 399, 1, 1.303},
    {35, 1e-12, 6, 30000, 137, 1, 0.826}, {35, 1e-12, 6, 30000, 231, 1, 1.222},
    {35, 1e-12, 6, 30000, 399, 1, 1.695}, {35, 1e-12, 8, 30000, 137, 1, 1.010},
    {35, 1e-12, 8, 30000, 231, 1, 1.506}, {35, 1e-12, 8, 30000, 399, 1, 2.106},
};

static void check_pairs_rule() {
  for (const Row& r : kRows) {
    BinLayout B;
    CHECK(layout(r.W, r.p, r.eps, r.W, 1e-3, B), "layout");
    const bool bins = bins_over_pairs(B, r.W, r.p, r.M, r.n, r.gradient != 0);
    CHECK(bins ? r.ratio > 1.0 / 1.1 : r.ratio < 1.3, "W %d p %d M %d, %d neighbours, gradient %d: by bins %d, measured %.2f",
          r.W, r.p, r.M, r.n, r.gradient, bins, r.ratio);
  }
}

// The same for weights stored once per pair over sums by bins, with n / W springs
// closer than dt.
static const Row kStored[] = {
    {35, 1e-12, 8, 1000, 708, 0, 0.616}, {35, 1e-12, 8, 3000, 536, 0, 0.640}, {35, 1e-12, 8, 3000, 914, 0, 0.800},
    {35, 1e-12, 8, 3000, 1305, 0, 1.251}, {35, 1e-12, 8, 5000, 544, 0, 0.814},
    {35, 1e-12, 8, 10000, 553, 0, 0.972}, {35, 1e-12, 8, 10000, 880, 0, 1.247},
    {35, 1e-12, 8, 10000, 1446, 0, 1.900}, {35, 1e-12, 8, 30000, 559, 0, 1.434},
    {35, 1e-12, 8, 30000, 895, 0, 2.013}, {35, 1e-12, 8, 60000, 559, 0, 1.420},
    {35, 1e-12, 4, 1000, 708, 0, 0.739}, {35, 1e-12, 4, 3000, 536, 0, 0.541}, {35, 1e-12, 4, 3000, 914, 0, 0.655},
    {35, 1e-12, 4, 3000, 1305, 0, 1.069}, {35, 1e-12, 4, 5000, 544, 0, 0.700},
    {35, 1e-12, 4, 10000, 553, 0, 0.763}, {35, 1e-12, 4, 10000, 880, 0, 1.058},
    {35, 1e-12, 4, 10000, 1446, 0, 1.616}, {35, 1e-12, 4, 30000, 559, 0, 1.176},
    {35, 1e-12, 4, 30000, 895, 0, 1.651}, {35, 1e-12, 4, 60000, 559, 0, 1.150},
    {18, 1e-06, 8, 1000, 708, 0, 0.844}, {18, 1e-06, 8, 3000, 536, 0, 1.181}, {18, 1e-06, 8, 3000, 914, 0, 1.274},
    {18, 1e-06, 8, 3000, 1305, 0, 1.275}, {18, 1e-06, 8, 5000, 544, 0, 1.443},
    {18, 1e-06, 8, 10000, 553, 0, 1.615}, {18, 1e-06, 8, 10000, 880, 0, 1.958},
    {18, 1e-06, 8, 10000, 1446, 0, 2.072}, {18, 1e-06, 8, 30000, 559, 0, 2.336},
    {18, 1e-06, 8, 30000, 895, 0, 2.828}, {18, 1e-06, 8, 60000, 559, 0, 1.521},
    {18, 1e-06, 4, 1000, 708, 0, 0.753}, {18, 1e-06, 4, 3000, 536, 0, 1.097}, {18, 1e-06, 4, 3000, 914, 0, 1.187},
    {18, 1e-06, 4, 3000, 1305, 0, 1.147}, {18, 1e-06, 4, 5000, 544, 0, 1.330},
    {18, 1e-06, 4, 10000, 553, 0, 1.432}, {18, 1e-06, 4, 10000, 880, 0, 1.719},
    {18, 1e-06, 4, 10000, 1446, 0, 1.772}, {18, 1e-06, 4, 30000, 559, 0, 2.048},
    {18, 1e-06, 4, 30000, 895, 0, 2.452}, {18, 1e-06, 4, 60000, 559, 0, 1.105},
    {35, 1e-12, 8, 1000, 708, 1, 0.977}, {35, 1e-12, 8, 3000, 536, 1, 0.986},
    {35, 1e-12, 8, 10000, 553, 1, 1.142}, {35, 1e-12, 8, 20000, 558, 1, 1.207},
    {35, 1e-12, 4, 1000, 708, 1, 0.898}, {35, 1e-12, 4, 3000, 536, 1, 0.896},
    {35, 1e-12, 4, 10000, 553, 1, 0.982}, {35, 1e-12, 4, 20000, 558, 1, 1.033},
    {18, 1e-06, 8, 1000, 708, 1, 1.158}, {18, 1e-06, 8, 3000, 536, 1, 1.089},
    {18, 1e-06, 8, 10000, 553, 1, 1.297}, {18, 1e-06, 8, 20000, 558, 1, 1.358},
};

static void check_stored_rule() {
  for (const Row& r : kStored) {
    BinLayout B;
    CHECK(layout(r.W, r.p, r.eps, r.W, 1e-3, B), "layout");
    const bool bins = bins_over_once(B, r.W, r.p, r.M, r.n, (double)r.n / r.W, r.gradient != 0);
    CHECK(bins ? r.ratio > 1.0 / 1.1 : r.ratio < 1.3, "W %d p %d M %d, %d neighbours, gradient %d: by bins %d, measured %.2f",
          r.W, r.p, r.M, r.n, r.gradient, bins, r.ratio);
  }
}

// Batches of equal instances by the library's choice (W = 35, p = 8), stored over by
// bins; and weights on the fly beside them, which share the launch.
static void check_batch_rule() {
  struct {
    int n, M, neighbours;
    double ratio;
  } rows[] = {{1, 600, 450, 0.84}, {2, 600, 450, 0.82}, {8, 600, 450, 1.06}, {64, 600, 450, 1.0}, {1, 3000, 434, 0.82},
              {4, 3000, 434, 0.97}, {16, 3000, 434, 1.11}, {1, 10000, 446, 0.88}, {4, 10000, 446, 1.18},
              {1, 1000, 705, 1.02}, {4, 1000, 705, 1.22}, {16, 1000, 705, 1.61}};
  BinLayout B;
  CHECK(layout(35, 8, 1e-12, 35, 1e-3, B), "layout");
  for (const auto& r : rows) {
    const double springs = (double)r.n * r.M;
    const BatchBins b = batch_bins(B, 35, springs, springs * r.neighbours, 0.0, 0.0);
    CHECK(!b.on_the_fly && (b.choice ? r.ratio > 1.0 / 1.1 : r.ratio < 1.1), "%d instances of %d, %d neighbours: by bins %d",
          r.n, r.M, r.neighbours, b.choice);
  }
  const BatchBins none = batch_bins(B, 35, 0.0, 0.0, 0.0, 0.0);
  CHECK(!none.choice && !none.on_the_fly, "an empty batch");
  CHECK(!batch_bins(B, 35, 0.0, 0.0, 300.0, 300.0 * 116).on_the_fly, "a few springs on the fly");
  CHECK(batch_bins(B, 35, 0.0, 0.0, 12000.0, 12000.0 * 127).on_the_fly, "many springs on the fly");
  const BatchBins both = batch_bins(B, 35, 450.0, 450.0 * 450, 129.0, 129.0 * 129);
  CHECK(both.choice && both.on_the_fly, "one launch for both groups");
}

// Blocks of the pair-once sum: of a plan and of a batch alike, few rows are spread
// over as many blocks as they can be.
static void check_rows() {
  CHECK(sym_rows(1, 1.0) == 8 && sym_rows(600, 450.0) == 8 && sym_rows(8191, 100.0) == 8, "few rows");
  CHECK(sym_rows(20000, 987.0) == 8 && sym_rows(60000, 1984.0) == 8, "long ranges");
  CHECK(sym_rows(10000, 138.0) == 16 && sym_rows(100000, 101.0) == 16, "many rows of short ranges");
}

// Sweeps of the solve: measured, us, by wavefronts, 64 and 16 rows a block.
static void check_sweeps() {
  struct {
    int M, nearby;
    double wave, r64, r16;
  } rows[] = {{300, 160, 2.92, 7.09, 4.89},    {1000, 24, 2.58, 3.38, 3.77},    {1000, 320, 3.40, 11.23, 5.24},
              {2000, 160, 3.19, 6.29, 4.91},   {2000, 640, 5.07, 19.71, 8.14},  {4000, 40, 3.10, 3.60, 4.15},
              {4000, 640, 8.21, 19.63, 8.12},  {4000, 1300, 14.96, 47.05, 13.99}, {8000, 24, 3.69, 3.39, 5.23},
              {8000, 160, 4.81, 6.54, 6.46},   {8000, 1300, 20.77, 50.50, 18.43}, {16000, 24, 5.56, 3.47, 7.73},
              {16000, 160, 8.70, 7.46, 10.38}, {16000, 640, 22.73, 28.91, 20.17}, {30000, 40, 8.77, 5.10, 16.10},
              {30000, 160, 16.93, 10.06, 17.88}, {30000, 1300, 107.82, 68.05, 58.39}, {60000, 80, 23.13, 11.13, 30.18},
              {200000, 320, 198.22, 98.25, 122.53}};
  for (const auto& r : rows) {
    const int form = sweep_rows(r.M, r.nearby);
    const double got = form == kSweepByRow ? r.wave : (form == 64 ? r.r64 : r.r16);
    CHECK(got <= 1.15 * std::min(r.wave, std::min(r.r64, r.r16)), "M %d, %d nearby: %d rows, %.2f us", r.M, r.nearby, form, got);
  }
}

int main() {
  check_rows();
  check_sweeps();
  check_batch_rule();
  check_look_up();
  check_pairs_rule();
  check_stored_rule();
  if (failures) return 1;
  std::printf("form checks passed\n");
  return 0;
}
