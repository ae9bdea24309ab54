// Index arithmetic of the sums by distance bins, shared by the kernels and the
// host (which checks it over the whole range of its arguments).
#pragma once

#include <math.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define WFP_HD __host__ __device__ __forceinline__
#else
#define WFP_HD inline
#endif

namespace wfp {

// Place of distance |z| in a chunk's lookup cells c0 .. c0 + ctop of width
// 1 / scale: the nearest one for distances outside the chunk.  Cut off before the
// conversion to int, whose range z scale leaves where a block of sources reaches
// across the box (1.1 at a step of 2e-7) and for missing sources (1e30 away, or
// 2 pi less that across the seam).
WFP_HD int bin_cell(double z, double scale, int c0, int ctop) {
  const int c = (int)fmin(fabs(z) * scale, (double)(c0 + ctop)) - c0;
  return c > 0 ? c : 0;
}

// What a window leaves to spare: a share of the step, and the rounding of the
// coordinates a turn apart (4 units in the last place of 2 pi), which outweighs
// it below steps of 1e-6.
WFP_HD double bin_tol(double dt) { return 1e-9 * dt + 4e-15; }

// Unwrapped target indices [l0, l1) below and [r0, r1) above a block's sources.
struct BinWindow {
  int l0, l1, r0, r1;
};

// Targets whose distance to some source in [xa, xb] may lie in [elo, ehi), with
// `tol` to spare; where both runs meet (and in the first chunk, which has the
// sources themselves) the lower one is empty.  Unwrapped: in the periodic box
// the coordinate of index u is xs[u mod M] + 2 pi floor(u / M), u in [-M, 2M).
WFP_HD BinWindow bin_window(const double* xs, int M, bool periodic, double xa, double xb, double elo, double ehi,
                            double tol, bool first) {
  constexpr double turn = 6.28318530717958647692;
  // first unwrapped index at or above coordinate v
  auto lower = [&](double v) {
    int lo = periodic ? -M : 0, hi = periodic ? 2 * M : M;
    while (lo < hi) {
      const int mid = lo + (hi - lo) / 2;
      const double x = mid < 0 ? xs[mid + M] - turn : (mid >= M ? xs[mid - M] + turn : xs[mid]);
      if (x < v) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  BinWindow w;
  w.l0 = lower(xa - ehi - tol);
  w.l1 = lower(xb - elo + tol);
  w.r0 = lower(xa + elo - tol);
  w.r1 = lower(xb + ehi + tol);
  if (first || w.r0 < w.l1) {
    w.r0 = w.l0;
    w.l1 = w.l0;
  }
  return w;
}

}  // namespace wfp
