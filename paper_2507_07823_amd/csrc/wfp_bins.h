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

// Place of distance z in a chunk's lookup cells c0 .. c0 + ctop of width
// 1 / scale: the nearest one for distances outside the chunk.  Cut off above
// before the conversion to int, which z scale exceeds where a block of sources
// reaches across the box (1.1 at a step of 2e-7) and for missing sources.
WFP_HD int bin_cell(double z, double scale, int c0, int ctop) {
  const int c = (int)fmin(z * scale, (double)(c0 + ctop)) - c0;
  return c > 0 ? c : 0;
}

}  // namespace wfp
