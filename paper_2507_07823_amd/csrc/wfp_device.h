// Small device functions shared by the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wfp {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 6.28318530717958647692;
constexpr double kInvTwoPi = 0.15915494309189533577;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Chebyshev series a_0/2 + sum a_k T_k(s) by Clenshaw
__device__ __forceinline__ double cheb(const double* __restrict__ a, int n, double s) {
  double b1 = 0.0, b2 = 0.0;
  for (int k = n - 1; k >= 1; --k) {
    const double b0 = fma(2.0 * s, b1, a[k] - b2);
    b2 = b1;
    b1 = b0;
  }
  return fma(s, b1, 0.5 * a[0] - b2);
}

__device__ __forceinline__ int mod_slot(int64_t n, int N) {
  int s = (int)(n % N);
  return s < 0 ? s + N : s;
}

// XCD-aware block order: consecutive hardware block ids go round-robin over
// the 8 XCDs; give each XCD a contiguous range of logical blocks so rows that
// share density history share an L2.  A bijection when nblocks % 8 == 0.
__device__ __forceinline__ int xcd_block(int b, int nblocks) {
  const int per = (nblocks + 7) >> 3;
  return (b & 7) * per + (b >> 3);
}

}  // namespace

}  // namespace wfp
