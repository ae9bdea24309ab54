// Which form the local sum takes: the layout of the distance bins, and the
// rules that choose between sums by bins, pair by pair and from stored weights.
// Pure C++, no HIP.
#pragma once

#include <array>
#include <cstdint>
#include <vector>

namespace wfp {

// Distance bins of the local sum (the kernels are in wfp_bins.hip): bins per
// chunk, lookup cells per chunk, the most lags (13 steps of 4) and bins.  With
// one quadrature node per lag of the window the bins end at W = 36.
constexpr int kBinChunk = 64, kBinCells = 4096, kMaxBinLags = 52, kMaxBins = 768;

// The bins of a window and a quadrature rule: edges (units of dt and distances,
// padded to whole chunks), lookup cells and chunks; the kernel's steps of four
// lags and the most edges within a cell.
struct BinLayout {
  int nbins = 0, nch = 0, ks = 0, bumps = 0;
  std::vector<double> D, edge, scales;
  std::vector<std::array<int, 4>> chunk;      // first cell, cells, their place, first steps of the halves
  std::vector<unsigned char> cells;
};

// Of a window of W steps of dt and parameter b, order p and quadrature nodes
// glz; false where they do not fit the kernel's limits.
bool bin_layout(int W, int p, double b, double dt, const std::vector<double>& glz, BinLayout& B);

// Microseconds of a level's local sum with the weights on the fly, for so many
// springs in the launch and neighbours a spring on average.
double bins_us(const BinLayout& B, double springs, double neighbours);
double pairs_us(int W, int p, double springs, double neighbours);

// No plan with fewer neighbours a spring takes bins.
constexpr double kBinNeighbours = 112.0;

// Whether weights on the fly are summed by bins; `gradient`: of a plan that
// keeps levels for gradients.
bool bins_over_pairs(const BinLayout& B, int W, int p, double springs, double neighbours, bool gradient);

// Microseconds of a level's local sum with the weights stored once per unordered
// pair, and whether local_mode 0 takes bins in its place; `nearby`: springs closer
// than dt on average.
double once_us(int W, int p, double springs, double neighbours);
bool bins_over_once(const BinLayout& B, int W, int p, double springs, double neighbours, double nearby, bool one_stream);

// The forms of a batch's instances that may go by bins: those whose mode is the
// library's choice (stored once per pair otherwise) and those with weights on the
// fly (pair by pair otherwise), each as one group.  W: the longest window; B: the
// layout of most chunks.
constexpr double kBatchBinNeighbours = 400.0;   // of the first group's instances, a spring
struct BatchBins {
  bool choice, on_the_fly;
};
BatchBins batch_bins(const BinLayout& B, int W, double choice_springs, double choice_pairs, double otf_springs,
                     double otf_pairs);

// Rows per block (of 8 wavefronts) of the pair-once stored local sum, by all the rows
// of a launch and their neighbours: one per wavefront, or two for many rows of short
// ranges, whose sources' values then serve twice the rows.  Levels, 16 / 8 rows: M = 1e4
// with 138 neighbours beside the history chain 53.8 / 56.5 us, 6e4 with 201 366 / 365, 3e4
// with 300 297 / 288, 994 861 / 792, 6e4 with 798 1379 / 1316, 1984 3246 / 3091; a gradient
// at 2e4 and 987 neighbours 1403 / 1342, 1349 before the values were staged; a batch of
// one instance of M = 600 with 450 106 / 88.  32 rows do not pay: M = 3e4 with 400, 406 us
// for 378.
inline int sym_rows(int64_t rows, double neighbours) { return rows >= 16 * 512 && neighbours < 256.0 ? 16 : 8; }

// Rows per block of the solve's global sweeps: 64 or 16 with the coupling stored once
// per pair, by diagonals, or kSweepByRow: a wavefront per row, from a row's values and
// columns.  A sweep of few rows is a chain of latencies, of which the last has the
// fewest, as long as its 12 bytes an entry stay in the L2 (30 MB); of many it is the
// stream of the values, of which the diagonals need a third; 16 rows where long runs
// would leave blocks of 64 too few.  One sweep, us, wavefronts / 64 / 16 rows: M = 2e3
// and 40 nearby springs 2.7 / 3.8 / 4.3, 160: 3.2 / 6.3 / 4.9, 640: 5.1 / 19.7 / 8.1; 8e3 and
// 80 4.3 / 4.9 / 6.2, 320: 6.8 / 11.0 / 6.9, 640: 12.4 / 19.5 / 11.3; 1.6e4 and 40 5.6 / 3.8 /
// 9.5, 320: 14.5 / 10.5 / 10.8, 640: 22.7 / 28.9 / 20.2; 3e4 and 80 12.2 / 7.0 / 17.5, 320: 24.8
// / 20.4 / 19.5; 2e5 and 80 69 / 31 / 96.
constexpr int kSweepByRow = 1;
inline int sweep_rows(int64_t M, double nearby) {
  if (M <= 8192 && nearby * (double)M <= 2.5e6) return kSweepByRow;
  return M < 32768 && nearby > 300.0 ? 16 : 64;
}

}  // namespace wfp
