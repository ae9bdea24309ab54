// Layout of the distance bins, and the rules that choose the local sum's form.
#include "wfp_forms.h"

#include <algorithm>
#include <cmath>

#include "wfp_host.h"

namespace wfp {

bool bin_layout(int W, int p, double b, double dt, const std::vector<double>& glz, BinLayout& B) {
  const int NQ = W + p / 2;
  const double delta = W * dt;
  B = BinLayout();
  // (a window of up to p / 2 steps has no room for an intermediate pair's stencil above
  // lag 0; the sums pair by pair let it start there, at the upper end's clamp)
  if (p > 8 || NQ > kMaxBinLags || W <= p / 2) return false;
  // bin width: 0.1 dt leaves the degree-7 polynomials of the default window
  // (b / W = 0.79) and p <= 8 within 1.4e-16 of the weights (p = 10 and 12 need
  // more terms); a steeper window takes narrower bins
  const double hmax = 0.1 * std::min(1.0, W / b * (27.631 / 35.0));
  B.D = bin_edges(W, p, glz, hmax);
  std::vector<double>&D = B.D, &edge = B.edge, &scales = B.scales;
  auto& chunk = B.chunk;
  std::vector<unsigned char>& cells = B.cells;
  B.nbins = (int)D.size() - 1;
  B.nch = (B.nbins + kBinChunk - 1) / kBinChunk;
  const int npad = B.nch * kBinChunk;
  if (npad > kMaxBins) return false;
  D.resize(npad + 1, D.back());
  edge.assign(npad + 1, delta);
  for (int i = 0; i < B.nbins; ++i) edge[i] = D[i] * dt;
  // lookup cells of a chunk: as narrow as its narrowest bin (then a cell holds
  // one edge at most) while they fit in kBinCells; at each cell's start the
  // record (0 below the chunk, then one per bin), four to a word
  scales.resize(B.nch);
  chunk.resize(B.nch);
  for (int c = 0; c < B.nch; ++c) {
    const double* e = &edge[c * kBinChunk];
    const int n = std::min(kBinChunk, B.nbins - c * kBinChunk);   // padding bins are empty
    double narrow = delta;
    for (int i = 0; i < n; ++i) narrow = std::min(narrow, e[i + 1] - e[i]);
    const double sc = scales[c] = std::min(1.01 / narrow, (kBinCells - 8) / (e[n] - e[0]));
    auto record = [&](double v) {
      const int r = (int)(std::upper_bound(e, e + n + 1, v) - e);
      return r > n ? kBinChunk + 1 : r;
    };
    const int c0 = (int)std::floor(e[0] * sc) - 1, c1 = (int)std::floor(e[n] * sc) + 1;
    chunk[c] = {c0, c1 - c0 + 1, (int)(cells.size() / 4), 0};
    if (c1 - c0 + 1 > kBinCells) return false;
    for (int i = c0; i <= c1; ++i) {
      const int r0 = record(i / sc - 1e-12 * delta), r1 = record((i + 1) / sc + 1e-12 * delta);
      cells.push_back((unsigned char)r0);
      B.bumps = std::max(B.bumps, std::min(r1, n + 1) - r0);
    }
    while (cells.size() % 4) cells.push_back((unsigned char)(kBinChunk + 1));
  }
  B.ks = (NQ + 3) / 4 <= 10 && B.bumps <= 2 ? 10 : 13;
  if (B.bumps > 4) return false;
  // first lag with weight in each half of a chunk (the lowest node's stencil
  // at its lower edge), as steps of four lags
  const double amax = 0.5 * (1.0 + *std::max_element(glz.begin(), glz.end()));
  auto step0 = [&](int bin) {
    const double d = D[bin];
    return std::max(0, (int)std::floor(W - (W - d) * amax - 1e-6) - p / 2 + 1) / 4;
  };
  for (int c = 0; c < B.nch; ++c) chunk[c][3] = step0(c * kBinChunk) | step0(c * kBinChunk + kBinChunk / 2) << 16;
  return true;
}

// By bins a block of 32 springs takes about the same time whatever its
// neighbours; 256 blocks run side by side (one per compute unit: their LDS), in
// rounds.  Lags are taken in 10 steps of four, or in 13 by a kernel with twice
// the look-ups.  Measured (us, M = 2e3 / 2e4 / 1e5; model in brackets): 12 chunks
// and 10 steps 82 / 231 / 979 (84 / 237 / 1000), 11 chunks 78 / 222 / 930 (79 /
// 222 / 932), 4 chunks and 13 steps 46 / 126 / 526 (50 / 134 / 555), 2 chunks and
// 10 steps 24 / 62 / 248 (28 / 67 / 263).
double bins_us(const BinLayout& B, double springs, double neighbours) {
  const double rounds = std::ceil(springs / 8192.0);
  const double round = (8.2 + 5.7 * B.nch) * (B.ks > 10 ? 1.35 : 1.0) * (1.0 + neighbours / 9000.0);
  return 8.0 + rounds * round;
}

// Pair by pair a level costs its (pair, node, order) steps and a share for the
// shortest launches.  Measured at W = 35, 231 neighbours, p = 2 / 4 / 6 / 8 (us):
// M = 2e3 47 / 60 / 69 / 84 (43 / 56 / 69 / 82), 2e4 184 / 236 / 294 / 342 (168 /
// 220 / 271 / 323), 1e5 733 / 952 / 1167 / 1387 (726 / 948 / 1170 / 1392); below M
// = 2e3 no less than there (p = 8: 68 at M = 1e3 and 126 neighbours (62), 64 at 256
// and 162 (71)).
double pairs_us(int W, int p, double springs, double neighbours) {
  // with the neighbours, against 231 of them (at 105 to 137 the ranges of a
  // workgroup's rows take another step of 256 sources)
  static const double x[] = {0, 105, 112, 137, 177, 231, 301, 400, 520}, y[] = {0.15, 0.59, 0.69, 0.83, 0.90, 1.0, 1.28, 1.59, 2.0};
  const int last = 8;
  double f = y[last] + 0.0034 * (neighbours - x[last]);
  for (int i = 0; i < last; ++i)
    if (neighbours >= x[i] && neighbours < x[i + 1]) f = y[i] + (y[i + 1] - y[i]) * (neighbours - x[i]) / (x[i + 1] - x[i]);
  return (105.0 + W * (11.4 + 3.17 * p)) * f * std::max(0.058, 0.04 + 0.96e-5 * springs);
}

// The line lies where the two meet: at W = 35 by 112 neighbours for p = 8 from M =
// 7e3 on (measured 115 at 2e4 and 1e5) and 200 at 2e3 (210), for p = 4 by 240 (225
// to 242) and 360 (405), for p = 2 by 340 (335 to 357) and 510.  A gradient takes
// two more sums by bins in a pass of twice the blocks, against one pass pair by
// pair: there the lines lie 1.1 to 1.25 times as far out at M = 3e4 (136, 180, 273
// and 386 neighbours for p = 8, 6, 4 and 2), and closer than the march's at 2e3 (136,
// 237, 307 and 372), where that pass leaves the chip idle.
bool bins_over_pairs(const BinLayout& B, int W, int p, double springs, double neighbours, bool gradient) {
  // (short launches pair by pair are at their cheapest at 140 to 200 neighbours: 62 us
  // for 77 by bins at M = 3e3 and 159)
  if (!gradient && springs < 4096.0 && neighbours < 200.0) return false;
  const double share = !gradient ? 1.0 : (springs < 4096.0 ? 0.9 : 1.17);
  return neighbours >= kBinNeighbours && share * bins_us(B, springs, neighbours) <= pairs_us(W, p, springs, neighbours);
}

// Bound by the weights' stream (W / 2 + p lags a pair), or by a row's range on
// small problems.  Measured (model) at W = 35, p = 8: M = 600 and 416 neighbours 39
// us (41), 1e3 and 708 59 (54), 3e3 and 536 56 (58), 1e4 and 553 166 (163), 3e4 and
// 559 444 (465); p = 4 at 3e4 382 (395).
double once_us(int W, int p, double springs, double neighbours) {
  const double bytes = 8.0 * 0.5 * springs * neighbours * (0.5 * W + p);
  return std::max(22.0 + 0.045 * neighbours, 15.0 + bytes / 3.8e6);
}

// From 64 MB of weights on stored sums run beside the history chain, which then
// costs no time of its own (25 us); but where the springs closer than dt are so many
// (28) that the solve goes by global sweeps, the sweeps wait for compute units (25
// us the other way).  Gradients and callers who ask for it run on one stream.  Levels measured, stored over
// by bins, at W = 35 and p = 8: 0.80 at M = 3e3 and 914 neighbours, 1.25 at 1305; 0.81
// at 5e3 and 544; 0.97 at 1e4 and 553, 1.25 at 880; 1.43 at 3e4 and 559; p = 4: 0.76 at
// 1e4 and 553, 1.06 at 880; 1.18 at 3e4 and 559.
bool bins_over_once(const BinLayout& B, int W, int p, double springs, double neighbours, double nearby, bool one_stream) {
  const bool beside = !one_stream && 4.0 * springs * neighbours * (0.5 * W + p) >= 64.0 * 1024 * 1024;
  const double chain = !beside ? 0.0 : (nearby >= 28.0 ? -25.0 : 25.0);
  return neighbours >= 512.0 && 1.02 * bins_us(B, springs, neighbours) + chain <= once_us(W, p, springs, neighbours);
}

// The launches of a form take all its instances, so the groups are weighed
// together: every combination's sums, one after the other.  Batches of the
// library's choice at W = 35, stored over by bins, us a level: one instance of M = 600
// with 450 neighbours 108 / 128, 64 of them 757 / 759; M = 3000 with 434: one 105 / 129,
// 4 220 / 228, 16 657 / 594; one of 1e4 with 446 197 / 223, 4 559 / 474; 16 of 1000 with
// 705 490 / 304.
BatchBins batch_bins(const BinLayout& B, int W, double choice_springs, double choice_pairs, double otf_springs,
                     double otf_pairs) {
  BatchBins best{false, false};
  double least = 0.0;
  for (int k = 0; k < 4; ++k) {
    const BatchBins b{(k & 1) != 0, (k & 2) != 0};
    if ((b.choice && choice_springs == 0.0) || (b.on_the_fly && otf_springs == 0.0)) continue;
    const double springs = (b.choice ? choice_springs : 0.0) + (b.on_the_fly ? otf_springs : 0.0);
    const double pairs = (b.choice ? choice_pairs : 0.0) + (b.on_the_fly ? otf_pairs : 0.0);
    double us = springs > 0.0 ? bins_us(B, springs, pairs / springs) : 0.0;
    if (!b.choice && choice_springs > 0.0) us += once_us(W, 8, choice_springs, choice_pairs / choice_springs);
    if (!b.on_the_fly && otf_springs > 0.0) us += pairs_us(W, 8, otf_springs, otf_pairs / otf_springs);
    if (k == 0 || us < least) {
      least = us;
      best = b;
    }
  }
  return best;
}

}  // namespace wfp
