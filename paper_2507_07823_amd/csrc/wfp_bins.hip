// Local sum by distance bins: the weights on the fly for springs with many
// neighbours.
//
// Q_m(d) (Section 4.1) depends on the distance alone and is piecewise smooth:
// its quadrature nodes s_i(d) are linear in d, and the stencils are fixed
// between the distances at which some s_i crosses a lag.  Those distances cut
// [0, delta) into bins (host: bin_edges), and on bin b
//   Q_m(d) = sum_k C[b][k][m] (d - e_b)^k,  k = 0 .. 7,
// to rounding.  So a pair's share of target j's sum,
//   sum_m Q_m(d) sigma_l^{L-m} = sum_k G_l[b][k] (d - e_b)^k,
//   G_l[b][k] = sum_m C[b][k][m] sigma_l^{L-m},
// is one polynomial of degree 7 whose coefficients depend on the source and
// the bin only: a product of the table C with the density history (matrix
// cores), then eight multiply-adds per ordered pair.
#include <type_traits>

#include "wfp_bins.h"
#include "wfp_device.h"
#include "wfp_kernels.h"

namespace wfp {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

// Position of the coefficient of (bin, k, lag m) in the table: the order in
// which the lanes of k_local_bins hold the matrix core's left operand.  Two
// bins make one tile of 16 rows; row g + 4 r of a tile comes back in element
// r of the lanes 16 g .. 16 g + 15, so that a lane's four results are four
// consecutive coefficients of one bin.
__device__ __forceinline__ int64_t bin_coef_pos(int bin, int k, int m, int ks) {
  const int g = (bin & 1) * 2 + (k >> 2), r = k & 3;
  return ((int64_t)(bin >> 1) * ks + (m >> 2)) * 64 + (g + 4 * r) + 16 * (m & 3);
}

// Unevaluated sums hi + lo of two doubles (error-free additions and products):
// a bin's power coefficients come from its values by divided differences that
// cancel five digits.
struct dd {
  double hi, lo;
};
__device__ __forceinline__ dd dd_norm(double a, double b) {
  const double s = a + b;
  return {s, b - (s - a)};
}
__device__ __forceinline__ dd dd_add(dd a, dd b) {
  const double s = a.hi + b.hi, v = s - a.hi;
  const double e = (a.hi - (s - v)) + (b.hi - v);
  return dd_norm(s, e + (a.lo + b.lo));
}
__device__ __forceinline__ dd dd_mul(dd a, double b) {
  const double p = a.hi * b;
  return dd_norm(p, fma(a.lo, b, fma(a.hi, b, -p)));
}
__device__ __forceinline__ dd dd_div(dd a, double b) {
  const double q = a.hi / b;
  return dd_norm(q, (fma(-q, b, a.hi) + a.lo) / b);
}

}  // namespace

// The table C, one bin per workgroup of 64 threads: Q_m at the 8 Chebyshev
// points of the bin (thread = point, share of the quadrature nodes), then the
// coefficients of the interpolating polynomial (thread = lag; Newton's form,
// expanded, in twice the working precision).  D: bin edges in units of dt.
// deriv: of (1/2) dQ_m/dd instead, with lag 0.
template <int P>
__global__ void __launch_bounds__(64)
k_bin_table(int nbins, int W, int NQ, int ks, int ngl, double dt, const double* __restrict__ D,
            const double* __restrict__ glz, const double* __restrict__ glw, const double* __restrict__ cheb_phi,
            const double* __restrict__ cheb_g, int ncheb, const double* __restrict__ lagw, int deriv,
            double* __restrict__ C) {
  __shared__ double acc[8][8][kMaxBinLags];
  const int bin = blockIdx.x;
  if (bin >= nbins) return;
  const int pt = threadIdx.x & 7, grp = threadIdx.x >> 3;
  const double lo = D[bin], hi = D[bin + 1], mid = 0.5 * (lo + hi);
  for (int m = 0; m < NQ; ++m) acc[pt][grp][m] = 0.0;
  const double x = lo + (hi - lo) * (0.5 + 0.5 * cos(kPi * (pt + 0.5) / 8.0));
  const int mmin = mid < 1.0 ? 0 : 1;
  for (int q = grp; q < ngl; q += 8) {
    const double a = 0.5 * (1.0 + glz[q]);
    // the bin's stencil of this node, from its middle
    int m0 = (int)floor(W - (W - mid) * a) - P / 2 + 1;
    m0 = max(mmin, min(m0, W - P / 2));
    const double s = W - (W - x) * a;
    const double rest = 1.0 - cheb(cheb_phi, ncheb, 2.0 * s / W - 1.0);
    const double half = 0.5 * (W - x) * glw[q], om = half * rest;
    const double u = s - m0;
    double pre[P], dpre[P];
    pre[0] = 1.0;
    dpre[0] = 0.0;
#pragma unroll
    for (int r = 1; r < P; ++r) {
      dpre[r] = dpre[r - 1] * (u - (r - 1)) + pre[r - 1];
      pre[r] = pre[r - 1] * (u - (r - 1));
    }
    // Q_m / dt, or (1/2) dQ_m/dd
    const double dom = deriv ? -0.5 * glw[q] * rest - half * a * (2.0 / W) * cheb(cheb_g, ncheb, 2.0 * s / W - 1.0) : 0.0;
    double suf = 1.0, dsuf = 0.0;
#pragma unroll
    for (int r = P - 1; r >= 0; --r) {
      const double v = lagw[r] * pre[r] * suf;
      const double dv = lagw[r] * (dpre[r] * suf + pre[r] * dsuf);
      acc[pt][grp][m0 + r] += deriv ? 0.5 * (dom * v + om * a * dv) : om * v;
      dsuf = dsuf * (u - r) + suf;
      suf *= (u - r);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 8 * NQ; e += 64) {
    const int m = e >> 3, p = e & 7;
    double v = 0.0;
    for (int g = 0; g < 8; ++g) v += acc[p][g][m];
    acc[p][0][m] = v;
  }
  __syncthreads();
  const double iw = 1.0 / ((hi - lo) * dt);
  // (lag 0 belongs to the implicit solve, except in the derivative)
  for (int m = (deriv ? 0 : 1) + (int)threadIdx.x; m < NQ; m += 64) {
    double t[8];
    dd f[8], c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      t[i] = 0.5 + 0.5 * cos(kPi * (i + 0.5) / 8.0);
      f[i] = {acc[i][0][m], 0.0};
      c[i] = {0.0, 0.0};
    }
#pragma unroll
    for (int j = 1; j < 8; ++j)
#pragma unroll
      for (int i = 7; i >= j; --i) f[i] = dd_div(dd_add(f[i], {-f[i - 1].hi, -f[i - 1].lo}), t[i] - t[i - j]);
    c[0] = f[7];
#pragma unroll
    for (int i = 6; i >= 0; --i) {   // c <- c (x - t_i) + f_i
#pragma unroll
      for (int k = 7 - i; k >= 1; --k) c[k] = dd_add(c[k - 1], dd_mul(c[k], -t[i]));
      c[0] = dd_add(f[i], dd_mul(c[0], -t[i]));
    }
    double w = deriv ? 1.0 : dt;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      C[bin_coef_pos(bin, k, m, ks)] = (c[k].hi + c[k].lo) * w;
      w *= iw;
    }
  }
}

#define WFP_BIN_TABLE(PP)                                                                                       \
  template __global__ void k_bin_table<PP>(int, int, int, int, int, double, const double*, const double*,       \
                                           const double*, const double*, const double*, int, const double*,      \
                                           int, double*);
WFP_BIN_TABLE(2)
WFP_BIN_TABLE(4)
WFP_BIN_TABLE(6)
WFP_BIN_TABLE(8)
#undef WFP_BIN_TABLE

// Target windows.  Block b holds nsrc consecutive sources; chunk
// c the distances [edge[c kBinChunk], edge[(c + 1) kBinChunk)).  win[b nch + c]
// = (l0, l1, r0, r1): every target within the chunk of some source of the block
// has its unwrapped index in [l0, l1) (below) or [r0, r1) (above).  span[b] =
// [l0, r1) of the last chunk, which holds them all.
__global__ void k_bin_windows(int M, int nsrc, int nblk, int nch, int periodic, double tol, const double* __restrict__ xs,
                              const double* __restrict__ edge, int4* __restrict__ win, int2* __restrict__ span) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nblk * nch) return;
  const int b = e / nch, c = e - b * nch;
  const double xa = xs[(int64_t)b * nsrc], xb = xs[min((b + 1) * nsrc, M) - 1];
  const BinWindow w = bin_window(xs, M, periodic != 0, xa, xb, edge[c * kBinChunk], edge[(c + 1) * kBinChunk], tol, c == 0);
  win[e] = make_int4(w.l0, w.l1, w.r0, w.r1);
  if (c == nch - 1) span[b] = make_int2(w.l0, w.r1);
}

// One workgroup per block of kBinColumns consecutive sources.  Chunk by chunk
// of kBinChunk bins, its wavefronts form the coefficients G of the sources on
// the matrix cores (histories in LDS, the table from L2, a tile ahead) into
// LDS, then evaluate the targets in reach: kBinTargets of
// them side by side in a wavefront and 64 / kBinTargets sources at a time.
// The two phases are kept apart because FP64 matrix and vector instructions
// share the FP64 units: side by side each vector instruction waits for a whole
// matrix one.  A source has a record per bin and zero records on both sides,
// where pairs of other chunks land; a pair's record comes from a table of
// uniform cells (the record that holds the cell's start, then at most BUMPS
// edges within the cell).  A target's sum over the block grows in
// part[off[b] + (u - first)], chunk by chunk in a fixed order: the first chunk
// whose windows hold it stores, later ones add.
//
// Bound by the instructions of the visits (look-up and polynomial of a pair) and the
// products, one after the other, and by the chunks' staging and barriers between them.
// Clumped springs, M = 1e6 and 5763 neighbours / 2e4 and 116, us with the reduction:
// 14506 / 228; without the products 10682 / 123, without the visits 8308 / 211, with
// constants for the records' reads 14135 / 225.  Pair by pair 250 ms / 236 us.
//
// H = 2: the two derivative sums of the gradient pass in one visit of the
// pairs, for half as many sources: weights (1/2) dQ_m/dd sign(x_j - x_l) with
// lag 0, on the levels r1 - m of a linear buffer (forward densities) into part
// and on the ring (adjoint ones) into part2.
template <int KS, int BUMPS, int H>
__device__ __forceinline__ void local_bins_body(int M, int NH, int NQ, int64_t L, const BinArgs& A,
                                                const double* __restrict__ xs, const double* __restrict__ hist,
                                                const double* __restrict__ lin, int64_t r1, int b) {
  // columns of G: sources, or sources x histories
  constexpr int S = kBinColumns, CB = kBinChunk, R = kBinRecords, TL = kBinTargets, PH = 64 / TL;
  constexpr int SRC = S / H, NS = SRC / PH, mfirst = H == 2 ? 0 : 1;
  constexpr int kWaves = kBinThreads / 64;          // two row tiles (of two bins) each per chunk
  static_assert(CB == 4 * kWaves && CB + 2 <= R, "two tiles per wavefront, zero records on both sides");
  static_assert(R % 16 == 4 && PH == 4, "the records of the four sources read at once fall on different banks");
  constexpr int kPlane = S * R * 2;                 // doubles of one coefficient pair's plane
  constexpr int kWords = (kBinCells / 4 + kBinThreads - 1) / kBinThreads;
  extern __shared__ double g[];                     // [4 pairs][S][R][2]
  __shared__ double2 eds[R], xsrc[SRC / 2];
  __shared__ double hl[4 * KS * S], scl[kMaxBins / CB];
  __shared__ int4 chs[kMaxBins / CB], wins[kMaxBins / CB];
  __shared__ unsigned cell[kBinCells / 4];
  const int nch = A.nch;
  const int4* __restrict__ win = A.win + (int64_t)b * nch;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j0 = b * SRC;
  // sources beyond M are out of reach
  if (threadIdx.x < SRC) {                          // source i PH + ph at place ph NS + i
    const int j = j0 + (threadIdx.x % NS) * PH + threadIdx.x / NS;
    ((double*)xsrc)[threadIdx.x] = j < M ? xs[j] : 1e30;
  }
  for (int i = threadIdx.x; i < 4 * S * R; i += kBinThreads)
    *(double2*)(g + 2 * (int64_t)i) = make_double2(0.0, 0.0);
  if ((int)threadIdx.x < nch) {
    chs[threadIdx.x] = A.chunk[threadIdx.x];
    scl[threadIdx.x] = A.scales[threadIdx.x];
    wins[threadIdx.x] = win[threadIdx.x];
  }
  // the sources' histories, lag by lag (the matrix core's right operand)
  const int slot0 = mod_slot(L, NH);
  for (int i = threadIdx.x; i < 4 * KS * S; i += kBinThreads) {
    const int m = i / S, j = j0 + i % SRC;
    const int slot = slot0 - m < 0 ? slot0 - m + NH : slot0 - m;
    const bool first = H == 2 && i % S < SRC;
    hl[i] = (m >= mfirst && m < NQ && j < M) ? (first ? lin[(r1 - m) * M + j] : hist[(int64_t)slot * M + j]) : 0.0;
  }
  // a row tile; lags below 4 K0 carry no weight in it.  Straight runs of
  // instructions for a few K0: the wavefronts feed their matrix core only while
  // nothing else holds up their issue.
  auto make = [&](auto k0, const double (&a)[KS], double* gr) {
    constexpr int K0 = decltype(k0)::value;
    const double* hp = hl + (lane >> 4) * S + (lane & 15);
    d4 acc[S / 16];
#pragma unroll
    for (int ct = 0; ct < S / 16; ++ct) acc[ct] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = K0; ks < KS; ++ks)
#pragma unroll
      for (int ct = 0; ct < S / 16; ++ct)
        acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], hp[4 * ks * S + 16 * ct], acc[ct], 0, 0, 0);
#pragma unroll
    for (int ct = 0; ct < S / 16; ++ct) {
      double* r = gr + 16 * ct * R * 2;
      *(double2*)r = make_double2(acc[ct][0], acc[ct][1]);
      *(double2*)(r + kPlane) = make_double2(acc[ct][2], acc[ct][3]);
    }
  };
  auto make_from = [&](int k0, const double (&a)[KS], double* gr) {
    if (k0 < kBinSkip) make(std::integral_constant<int, 0>{}, a, gr);
    else if (k0 < 2 * kBinSkip) make(std::integral_constant<int, kBinSkip>{}, a, gr);
    else if (k0 < 3 * kBinSkip) make(std::integral_constant<int, 2 * kBinSkip>{}, a, gr);
    else make(std::integral_constant<int, 3 * kBinSkip>{}, a, gr);
  };
  // this lane's part of a record of the wavefront's first tile
  double* g0 = g + ((lane >> 4) & 1) * 2 * kPlane + ((lane & 15) * R + 1 + 2 * wv + (lane >> 5)) * 2;
  const double* __restrict__ cl = A.C + (int64_t)wv * KS * 64 + lane;
  auto load = [&](double (&a)[KS], int tile) {
    const double* __restrict__ ct0 = cl + (int64_t)tile * KS * 64;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = ct0[ks * 64];
  };
  double a0[KS];
  load(a0, 0);
  const int ph = lane / TL;
  const int first = win[nch - 1].x;                 // lowest target of the block
  double* __restrict__ pb = A.part + A.off[b];
  double* __restrict__ pb2 = H == 2 ? A.part2 + A.off[b] : nullptr;
  // target of this lane in unit t of the windows w, and its coordinate (out of
  // reach where there is none)
  auto target = [&](const int4& w, int t, bool& valid) {
    const int nl = (w.y - w.x + TL - 1) / TL;
    const int u = (t < nl ? w.x + t * TL : w.z + (t - nl) * TL) + (lane & (TL - 1));
    valid = u < (t < nl ? w.y : w.w);
    return u;
  };
  auto place = [&](int u, bool valid) {
    const int uu = u < 0 ? u + M : (u >= M ? u - M : u);
    return valid ? xs[uu] : -1e30;
  };
  int4 prev = make_int4(0, 0, 0, 0);
  __syncthreads();                                  // the tables above are in place
  for (int c = 0; c < nch; ++c) {
    const int4 w = wins[c], ch = chs[c];            // ch: first cell, cells, their place in the table, two k0
    unsigned cv[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const int e = i * kBinThreads + (int)threadIdx.x;
      cv[i] = e < (ch.y + 3) / 4 ? A.cells[ch.z + e] : 0u;
    }
    // the ends of record r, bin c CB + r - 1
    double2 ev = make_double2(0.0, 1e300);
    if (threadIdx.x < R) {
      const int e = c * CB + (int)threadIdx.x - 1;
      if (e >= 0) ev.x = A.edge[min(e, nch * CB)];
      if (threadIdx.x <= CB) ev.y = A.edge[e + 1];
    }
    bool valid;
    int u = target(w, wv, valid);
    double x = place(u, valid);
    {
      double a1[KS];
      load(a1, c * (CB / 2) + kWaves);
      make_from(__builtin_amdgcn_readfirstlane(ch.w & 0xffff), a0, g0);
      make_from(__builtin_amdgcn_readfirstlane(ch.w >> 16), a1, g0 + kWaves * 4);
    }
#pragma unroll
    for (int i = 0; i < kWords; ++i)
      if (i * kBinThreads + (int)threadIdx.x < kBinCells / 4) cell[i * kBinThreads + threadIdx.x] = cv[i];
    if (threadIdx.x < R) eds[threadIdx.x] = ev;
    __syncthreads();                                // the chunk is ready
    const int c0 = ch.x, ctop = ch.y - 1;
    const double scale = scl[c];
    const unsigned char* cellb = (const unsigned char*)cell;
    const int nu = (w.y - w.x + TL - 1) / TL + (w.w - w.z + TL - 1) / TL;
    for (int t = wv; t < nu; t += kWaves) {
      // the next unit's coordinates, loaded ahead
      bool vnext;
      const int unext = target(w, t + kWaves, vnext);
      const double xnext = place(unext, vnext);
      const bool seen = valid && c > 0 && u >= prev.x && u < prev.w;
      double old[H] = {};
      if (seen && ph == 0) {
        old[0] = pb[u - first];
        if (H == 2) old[H - 1] = pb2[u - first];
      }
      // pairs across the periodic seam: 2 pi - |x - x_l|
      const bool wrap = valid && (u < 0 || u >= M);
      const bool anyw = __any(wrap);
      double sum[H] = {};
      auto visit = [&](auto seam) {
        // the records of four pairs, then their polynomials, two at a time
#pragma unroll 1
        for (int i0 = 0; i0 < NS; i0 += 4) {
          double z[4], sg[4];
          int rec[4];
          const double2* y = xsrc + (ph * NS + i0) / 2;
          z[0] = x - y[0].x;
          z[1] = x - y[0].y;
          z[2] = x - y[1].x;
          z[3] = x - y[1].y;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (H == 2) {                           // sign(x_j - x_l), the shorter way round
              sg[i] = z[i] == 0.0 ? 0.0 : copysign(1.0, z[i]);
              if (seam) sg[i] = wrap ? -sg[i] : sg[i];
            }
            z[i] = fabs(z[i]);
            if (seam) z[i] = wrap ? kTwoPi - z[i] : z[i];
            rec[i] = cellb[bin_cell(z[i], scale, c0, ctop)];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            double2 e = eds[rec[i]];
#pragma unroll
            for (int s = 0; s < BUMPS; ++s) {
              const bool up = z[i] >= e.y;
              rec[i] += up ? 1 : 0;
              if (s + 1 < BUMPS) e = eds[rec[i]];
              else e.x = up ? e.y : e.x;
            }
            z[i] -= e.x;
          }
#pragma unroll
          for (int k0 = 0; k0 < 4; k0 += 2) {
            // every pair in another chunk
            if (!__any((unsigned)(rec[k0] - 1) < (unsigned)CB || (unsigned)(rec[k0 + 1] - 1) < (unsigned)CB)) continue;
#pragma unroll
            for (int n = 0; n < H; ++n) {
              double2 q[2][4];
#pragma unroll
              for (int k = 0; k < 2; ++k) {
                const double* r = g + (((i0 + k0 + k) * PH + ph + n * SRC) * R + rec[k0 + k]) * 2;
#pragma unroll
                for (int o = 0; o < 4; ++o) q[k][o] = *(const double2*)(r + o * kPlane);
              }
              double v[2];
#pragma unroll
              for (int k = 0; k < 2; ++k) v[k] = fma(q[k][3].y, z[k0 + k], q[k][3].x);
#pragma unroll
              for (int o = 2; o >= 0; --o) {
#pragma unroll
                for (int k = 0; k < 2; ++k) v[k] = fma(v[k], z[k0 + k], q[k][o].y);
#pragma unroll
                for (int k = 0; k < 2; ++k) v[k] = fma(v[k], z[k0 + k], q[k][o].x);
              }
              if (H == 2) sum[n] = fma(sg[k0 + 1], v[1], fma(sg[k0], v[0], sum[n]));
              else sum[n] += v[0] + v[1];
            }
          }
        }
      };
      if (anyw) visit(std::true_type{});
      else visit(std::false_type{});
#pragma unroll
      for (int o = 32; o >= TL; o >>= 1)
#pragma unroll
        for (int n = 0; n < H; ++n) sum[n] += __shfl_xor(sum[n], o, 64);
      if (valid && ph == 0) {
        pb[u - first] = seen ? old[0] + sum[0] : sum[0];
        if (H == 2) pb2[u - first] = seen ? old[H - 1] + sum[H - 1] : sum[H - 1];
      }
      u = unext;
      valid = vnext;
      x = xnext;
    }
    prev = w;
    load(a0, (c + 1) * (CB / 2));                   // (the table ends in a spare chunk)
    __syncthreads();                                // the chunk is done with
  }
}

template <int KS, int BUMPS, int H>
__global__ void __launch_bounds__(kBinThreads, 4)
k_local_bins(int M, int NH, int NQ, int64_t L, BinArgs A, const double* __restrict__ xs,
             const double* __restrict__ hist, const double* __restrict__ lin, int64_t r1) {
  const int b = xcd_block(blockIdx.x, gridDim.x);
  if (b >= A.nblk) return;                          // padding block (uniform)
  local_bins_body<KS, BUMPS, H>(M, NH, NQ, L, A, xs, hist, lin, r1, b);
}

#define WFP_LOCAL_BINS(KS, BUMPS, H)                                                                             \
  template __global__ void k_local_bins<KS, BUMPS, H>(int, int, int, int64_t, BinArgs, const double*,             \
                                                      const double*, const double*, int64_t);
WFP_LOCAL_BINS(10, 1, 1)
WFP_LOCAL_BINS(10, 2, 1)
WFP_LOCAL_BINS(13, 4, 1)
WFP_LOCAL_BINS(10, 1, 2)
WFP_LOCAL_BINS(10, 2, 2)
WFP_LOCAL_BINS(13, 4, 2)
#undef WFP_LOCAL_BINS

// The same over (instance, block of sources) items of a batch.
__global__ void __launch_bounds__(kBinThreads, 4) kb_local_bins(BatchLaunch bl) {
  const int2 w = bl.work[xcd_block(blockIdx.x, gridDim.x)];
  if (w.x < 0) return;                              // block-uniform
  const InstDesc& d = bl.desc[w.x];
  if (*bl.level >= d.end) return;                   // the instance has marched its own levels (block-uniform)
  local_bins_body<10, 2, 1>(d.M, d.NH, d.NQ, *bl.level, d.bins, d.xs, d.hist, nullptr, 0, w.y);
}

// Row l's total: the sums that the blocks whose windows hold l (or, in the
// periodic box, l - M or l + M) wrote for it, in block order, scaled per row.
// A workgroup takes 64 consecutive rows, one per lane; cov[3 w + i] = the run
// [x, y) of blocks that may hold row range w's image i (l - M, l, l + M), cut
// into kReduceWaves consecutive parts, one per wavefront.
__device__ __forceinline__ void local_bins_reduce_body(int M, const BinArgs& A, const double* __restrict__ part,
                                                       const double* __restrict__ scale, double* __restrict__ out,
                                                       int bid) {
  __shared__ double tot[kReduceWaves][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int l = bid * 64 + lane;
  double acc = 0.0;
  for (int im = 0; im < 3; ++im) {
    const int2 r = A.cov[3 * bid + im];
    const int n = r.y - r.x;
    if (n <= 0) continue;
    const int u = l + (im - 1) * M;
    const int q0 = r.x + (int)((int64_t)wv * n / kReduceWaves), q1 = r.x + (int)((int64_t)(wv + 1) * n / kReduceWaves);
    for (int q = q0; q < q1; q += 4) {
      double v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[k] = 0.0;
        if (q + k < q1) {
          const int2 s = A.span[q + k];
          if (l < M && u >= s.x && u < s.y) v[k] = part[A.off[q + k] + (u - s.x)];
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += v[k];
    }
  }
  tot[wv][lane] = acc;
  __syncthreads();
  if (wv == 0 && l < M) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kReduceWaves; ++w) t += tot[w][lane];
    out[l] = scale[l] * t;
  }
}

__global__ void __launch_bounds__(64 * kReduceWaves)
k_local_bins_reduce(int M, BinArgs A, const double* __restrict__ part, const double* __restrict__ scale,
                    double* __restrict__ out) {
  local_bins_reduce_body(M, A, part, scale, out, blockIdx.x);
}

__global__ void __launch_bounds__(64 * kReduceWaves) kb_local_bins_reduce(BatchLaunch bl) {
  const int2 w = bl.work[blockIdx.x];
  if (w.x < 0) return;
  const InstDesc& d = bl.desc[w.x];
  if (*bl.level >= d.end) return;                   // the instance has marched its own levels (block-uniform)
  local_bins_reduce_body(d.M, d.bins, d.bins.part, d.half_beta, d.loc, w.y);
}

}  // namespace wfp
