// Output regridding: cross-sections computed on one resident grid resampled onto another,
// for results on a user grid of fixed resolving power (section "Similar tools": any user
// wavelength or wavenumber grid, which fixes the spectral resolution; closing paragraph of
// "Functionality of pyROX": results converted for other codes' grids).
//
// Each source row is read as the piecewise-linear function through its grid nodes, zero
// outside the source range. Two forms:
//   linear  : that function at each destination point;
//   bin mean: its mean over each destination point's bin. Bin k spans from the midpoint
//             with the previous destination point to the midpoint with the next one (the
//             first and last bins mirrored to the same half-widths), clipped to the source
//             range; a bin wholly outside the source range gives 0. The integral over a bin
//             is summed over the source intervals it covers (trapezoids, partial ones at
//             its ends), so bin means times bin widths add up to the integral of the
//             function over the bins' union.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "../../include/xsec.h"
#include "kernel_args.h"
#include "runtime_internal.h"

namespace xs {

// First i in [0, n) with x[i] > v (n if none).
__device__ __forceinline__ int64_t upper_index(const double* __restrict__ x, int64_t n,
                                               double v) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (x[mid] > v) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// The linear interpolant of (x, y) at v inside [x[0], x[n-1]], given i = upper_index(v).
__device__ __forceinline__ double interp_at(const double* __restrict__ x,
                                            const double* __restrict__ y, int64_t n,
                                            int64_t i, double v) {
  if (i >= n) return y[n - 1];   // v == x[n - 1]
  if (i == 0) return y[0];
  const double t = (v - x[i - 1]) / (x[i] - x[i - 1]);
  return y[i - 1] + t * (y[i] - y[i - 1]);
}

constexpr int kRegridBlock = 256;
constexpr int kRegridRows = 4;            // rows per unit of work
constexpr int64_t kRegridGrid = 1 << 18;  // most workgroups of a launch (units are strided)

// Bin of destination point k, clipped to the source range [lo, hi]: midpoints between
// neighbours, the end bins mirrored; a single point takes the whole source range. False when
// the bin is empty.
__device__ __forceinline__ bool bin_of(const double* __restrict__ dst_x, int64_t n_dst, int64_t k,
                                       double lo, double hi, double* a, double* b) {
  if (n_dst == 1) {
    *a = lo;
    *b = hi;
  } else {
    *a = k > 0 ? 0.5 * (dst_x[k - 1] + dst_x[k]) : dst_x[0] - 0.5 * (dst_x[1] - dst_x[0]);
    *b = k + 1 < n_dst ? 0.5 * (dst_x[k] + dst_x[k + 1])
                       : dst_x[k] + 0.5 * (dst_x[k] - dst_x[k - 1]);
  }
  *a = fmax(*a, lo);
  *b = fmin(*b, hi);
  return *b > *a;
}

// Linear interpolation: one thread per destination point and kRegridRows rows, so a point's
// interval is searched once for them.
__global__ __launch_bounds__(kRegridBlock) void xs_regrid_linear_kernel(
    const double* __restrict__ src_x, int64_t n_src, const double* __restrict__ src,
    const double* __restrict__ dst_x, int64_t n_dst, int64_t n_rows, int64_t n_units,
    double* __restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n_units; u += stride) {
    const int64_t part = u / n_dst, k = u - part * n_dst, r0 = part * kRegridRows;
    const double v = dst_x[k];
    const bool in = !(v < src_x[0] || v > src_x[n_src - 1]);
    const int64_t i = in ? upper_index(src_x, n_src, v) : 0;
#pragma unroll
    for (int r = 0; r < kRegridRows; ++r)
      if (r0 + r < n_rows)
        out[(r0 + r) * n_dst + k] = in ? interp_at(src_x, src + (r0 + r) * n_src, n_src, i, v)
                                       : 0.0;
  }
}

// The first index of [0, n) with x > va, and the first with x >= vb, by G lanes: every step
// cuts both ranges to a G-th (four dependent loads for 6e5 nodes by 64 lanes, not forty).
template <int G>
__device__ __forceinline__ void bin_search(const double* __restrict__ x, int64_t n, double va,
                                           double vb, int l, int first_lane, int64_t* ia,
                                           int64_t* ib) {
  if constexpr (G == 1) {
    *ia = upper_index(x, n, va);
    *ib = *ia;
    while (*ib < n && x[*ib] < vb) ++*ib;
    return;
  }
  int64_t lo[2] = {0, 0}, hi[2] = {n, n};
  const uint64_t mask = G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull;
  while (lo[0] < hi[0] || lo[1] < hi[1]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int64_t step = (hi[t] - lo[t] + G - 1) / G;
      const int64_t p = lo[t] + l * step + step - 1;
      bool up = true;
      if (step > 0 && p < hi[t]) up = t == 0 ? x[p] > va : x[p] >= vb;
      // (a lane past the end says true: the answer is at most hi)
      const uint64_t m = (__ballot(up) >> first_lane) & mask;
      const int f = m ? __builtin_ctzll(m) : G;
      if (step > 0) {
        const int64_t at = lo[t] + f * step;
        hi[t] = min(hi[t], at + step - 1);
        lo[t] = min(at, hi[t]);
      }
    }
  }
  *ia = lo[0];
  *ib = lo[1];
}

// Bin means, G lanes per bin and kRegridRows rows. The trapezoid sum over the pieces inside
// the bin gives every node the weight of half the distance of its neighbours (clipped to the
// bin), the same for all rows: the lanes take the bin's nodes in turn, so rows are read in
// whole lines of the cache and each weight is formed once. 12 rows of 6e5 points onto 3e3 bins
// take 30 us (2 TB/s: the two searches and the bin's ends are some ten dependent loads beside
// the rows' own); one thread per row and bin, each in a line of the cache of its own, took 187.
template <int G>
__global__ __launch_bounds__(kRegridBlock) void xs_regrid_mean_kernel(
    const double* __restrict__ src_x, int64_t n_src, const double* __restrict__ src,
    const double* __restrict__ dst_x, int64_t n_dst, int64_t n_rows, int64_t n_units,
    double* __restrict__ out) {
  constexpr int kAhead = G == 64 ? 4 : G == 16 ? 2 : 1;   // nodes a lane has in flight
  const int lane = threadIdx.x & 63, l = lane & (G - 1), first = lane - l;
  const int64_t stride = (int64_t)gridDim.x * (kRegridBlock / G);
  const double lo = src_x[0], hi = src_x[n_src - 1];
  for (int64_t u = ((int64_t)blockIdx.x * kRegridBlock + threadIdx.x) / G; u < n_units;
       u += stride) {
    const int64_t part = u / n_dst, k = u - part * n_dst, r0 = part * kRegridRows;
    const int nr = (int)min((int64_t)kRegridRows, n_rows - r0);
    double a, b;
    if (!bin_of(dst_x, n_dst, k, lo, hi, &a, &b)) {
      for (int r = l; r < nr; r += G) out[(r0 + r) * n_dst + k] = 0.0;
      continue;
    }
    // nodes strictly inside (a, b): [i0, i1)
    int64_t i0, i1;
    bin_search<G>(src_x, n_src, a, b, l, first, &i0, &i1);
    const double* y = src + r0 * n_src;
    double s[kRegridRows];
#pragma unroll
    for (int r = 0; r < kRegridRows; ++r) s[r] = 0.0;
    for (int64_t i = i0 + l; i < i1; i += kAhead * G) {
#pragma unroll
      for (int t = 0; t < kAhead; ++t) {
        const bool ok = t == 0 || i + t * G < i1;
        const int64_t j = ok ? i + t * G : i;
        const double x0 = j > i0 ? src_x[j - 1] : a, x1 = j + 1 < i1 ? src_x[j + 1] : b;
        const double w = 0.5 * (x1 - x0);
#pragma unroll
        for (int r = 0; r < kRegridRows; ++r) {
          const double f = fma(y[min(r, nr - 1) * n_src + j], w, s[r]);
          s[r] = ok ? f : s[r];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kRegridRows; ++r)
#pragma unroll
      for (int d = G / 2; d >= 1; d /= 2) s[r] += __shfl_xor(s[r], d);
    // the function at the bin's ends, the rows dealt to the lanes
    const int64_t ib = i1 < n_src && src_x[i1] == b ? i1 + 1 : i1;   // first node above b
    const double wa = 0.5 * ((i1 > i0 ? src_x[i0] : b) - a);
    const double wb = 0.5 * (b - (i1 > i0 ? src_x[i1 - 1] : a));
#pragma unroll
    for (int r = 0; r < kRegridRows; ++r) {
      if ((r & (G - 1)) != l || r >= nr) continue;
      const double* yr = y + r * n_src;
      const double ya = interp_at(src_x, yr, n_src, i0, a), yb = interp_at(src_x, yr, n_src, ib, b);
      out[(r0 + r) * n_dst + k] = (s[r] + ya * wa + yb * wb) / (b - a);
    }
  }
}

// Lanes per bin by the average number of nodes in one: enough that a lane has a few nodes,
// few enough that the search and the sums over lanes stay small beside them. Measured, 12
// rows of 6e5 or 3e4 points, with 1 / 4 / 16 / 64 lanes (us): 0.3 nodes per bin 12 / 37 / 102 /
// 391, 3.3: 11 / 10 / 17 / 49, 20: 180 / 45 / 52 / 191, 67: 367 / 55 / 29 / 65, 200: 990 /
// 113 / 29 / 30, 666: 2669 / 319 / 59 / 25.
static int bin_lanes(size_t n_src, size_t n_dst) {
  return n_src >= 200 * n_dst ? 64 : n_src >= 24 * n_dst ? 16 : 2 * n_src >= 5 * n_dst ? 4 : 1;
}

}  // namespace xs

using namespace xs;

extern "C" int xs_regrid(xs_ctx* c, xs_grid_t src_h, xs_grid_t dst_h, const double* sigma_src,
                         size_t n_rows, int mode, double* out, int on_device, void* stream) {
  if (!c || !sigma_src || !out) return fail(XS_EINVAL, "NULL argument");
  if (mode != XS_REGRID_LINEAR && mode != XS_REGRID_BIN_MEAN)
    return fail(XS_EINVAL, "unknown regrid mode %d", mode);
  if (n_rows == 0 || n_rows > ((size_t)1 << 20))
    return fail(XS_EINVAL, "n_rows must be in [1, 2^20] (got %zu)", n_rows);
  GridRes* S;
  GridRes* D;
  {
    std::lock_guard<std::mutex> lk(c->mu);
    S = c->find_grid(src_h);
    D = c->find_grid(dst_h);
  }
  if (!S || !D) return fail(XS_ENOTFOUND, "unknown source or destination grid");
  if (S->n < 2) return fail(XS_EINVAL, "the source grid needs at least 2 points");
  hipError_t e = hipSetDevice(c->device);
  if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  const size_t in_bytes = n_rows * S->n * sizeof(double);
  const size_t out_bytes = n_rows * D->n * sizeof(double);
  void* buf = nullptr;
  const double* src_dev = sigma_src;
  double* out_dev = out;
  if (!on_device) {
    const size_t in_al = (in_bytes + 255) & ~(size_t)255;
    int rc = c->dev_alloc_again(&buf, in_al + out_bytes, "regrid staging");
    if (rc) return rc;
    e = hipMemcpyAsync(buf, sigma_src, in_bytes, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) {
      c->dev_free(buf, in_al + out_bytes);
      return hip_fail(e, "regrid upload");
    }
    src_dev = (const double*)buf;
    out_dev = (double*)((char*)buf + in_al);
  }
  const int lanes = mode == XS_REGRID_LINEAR ? 1 : bin_lanes(S->n, D->n);
  const int64_t units = (int64_t)D->n * ((int64_t)(n_rows + kRegridRows - 1) / kRegridRows);
  const int64_t per = kRegridBlock / lanes;
  const dim3 grid((unsigned)std::min<int64_t>(kRegridGrid, (units + per - 1) / per));
  auto kernel = mode == XS_REGRID_LINEAR ? xs_regrid_linear_kernel
                : lanes == 1 ? xs_regrid_mean_kernel<1>
                : lanes == 4 ? xs_regrid_mean_kernel<4>
                : lanes == 16 ? xs_regrid_mean_kernel<16> : xs_regrid_mean_kernel<64>;
  hipLaunchKernelGGL(kernel, grid, dim3(kRegridBlock), 0, st, S->d, (int64_t)S->n, src_dev, D->d,
                     (int64_t)D->n, (int64_t)n_rows, units, out_dev);
  e = hipGetLastError();
  if (e == hipSuccess && !on_device) {
    e = hipMemcpyAsync(out, out_dev, out_bytes, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  if (buf) c->dev_free(buf, ((in_bytes + 255) & ~(size_t)255) + out_bytes);
  if (e != hipSuccess) return hip_fail(e, "regrid");
  return XS_OK;
}
