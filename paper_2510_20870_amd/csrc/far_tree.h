// Far field by moments of line groups: the lines in order of their centres form a tree of
// groups (kLeafLines lines per leaf, kArity children per node), and a group far from a grid
// point enters its sum as one short series instead of line by line.
//
// Outside the core, Re w(z) is the real part of i/sqrt(pi) E[1 / (z - t)], t Gaussian with
// variance 1/2 (its asymptotic expansion, term by term). For a line of strength S, centre
// nu0, Doppler width b and Lorentz width g the contribution at nu is therefore
//     S/pi Re E[ i / (X - (delta + b t)) ],  X = nu - c,  delta = (nu0 - c) - i g,
// about any real centre c, which expands in 1/X:
//     S/pi sum_m V_m / X^(m+1),   V_m = -Im T_m,   T_m = E[(delta + b t)^m],
//     T_0 = 1, T_1 = delta, T_(m+1) = delta T_m + m (b^2/2) T_(m-1).
// The sums over a group's lines of (S/pi) V_m / s^m, s = sqrt(h^2 + g_max^2) + beta b_max
// (h half the group's extent, c its middle), are its moments A_1 .. A_NM. They move to a
// parent's centre by the binomial theorem. At |X| >= theta s the series is within
// 5e-8 of every line's own contribution with 16 moments (theta 3.5, beta 2.05), and within
// 3e-14 with 28 (beta 2.35), measured against a reference Faddeeva routine over the whole
// range of h, g and b. All of it is FP64.
//
// Leaves of 16 lines, because the lines of the leaves around a point are summed one by one:
// a leaf's half extent enters the distance from which it counts as far 3.5-fold. Four
// children, because a level's nodes then serve distances up to four times its own.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_args.h"
#include "voigt.h"

namespace xs {

constexpr int kLeafLines = 16;       // one DPP row of lines
constexpr int kArityBits = 2;
constexpr int kArity = 1 << kArityBits;
constexpr double kFarTheta = 3.5;    // a group is far where |nu - c| >= kFarTheta * s
// moments of the FP32 and the FP64 path, and the weight of the Doppler width in s
constexpr int kMomFp32 = 16, kMomFp64 = 28;
constexpr double kBetaFp32 = 2.05, kBetaFp64 = 2.35;
template <int NM> constexpr double far_beta() { return NM == kMomFp32 ? kBetaFp32 : kBetaFp64; }

// A node's fields: centres of the group's first and last line, scale s, largest Lorentz
// width, smallest and largest cut (leaves only), moments. Nodes are stored eight by eight,
// field by field (kNodeBlock nodes of a field side by side), so that wavefronts reading one
// field of neighbouring nodes read whole lines of the cache; every level starts at a multiple
// of kNodeBlock.
constexpr int kNodeBlock = 8;
enum { kNodeLo, kNodeHi, kNodeS, kNodeG, kNodeCutMin, kNodeCutMax, kNodeA };
template <int NM> constexpr int node_fields() { return kNodeA + NM; }
constexpr size_t node_bytes(int moments) { return (size_t)(kNodeA + moments) * sizeof(double); }
template <int NM>
__host__ __device__ __forceinline__ int64_t node_pos(int64_t node) {
  return (node / kNodeBlock) * (kNodeBlock * node_fields<NM>()) + node % kNodeBlock;
}
template <int NM, class T>   // T: double or const double
struct NodeRef {
  T* p;
  __host__ __device__ __forceinline__ T& at(int f) const { return p[f * kNodeBlock]; }
  __host__ __device__ __forceinline__ double lo() const { return at(kNodeLo); }
  __host__ __device__ __forceinline__ double hi() const { return at(kNodeHi); }
  __host__ __device__ __forceinline__ double s() const { return at(kNodeS); }
  __host__ __device__ __forceinline__ double c() const { return 0.5 * (lo() + hi()); }
};
template <int NM>
__host__ __device__ __forceinline__ NodeRef<NM, const double> node_at(const double* nodes,
                                                                      const TreeDims& d, int l,
                                                                      int64_t q) {
  return {nodes + node_pos<NM>(d.off[l] + q)};
}

// Moments V_m (m = 1 .. NM, times w) of one line in units of the scale: d = (nu0 - c)/s,
// g = gamma/s, q = (b/s)^2 / 2.
template <int NM>
__host__ __device__ __forceinline__ void line_moments(double w, double d, double g, double q,
                                                      double (&A)[NM]) {
  double u0 = 1.0, v0 = 0.0, u1 = d, v1 = g;
  A[0] = w * v1;
#pragma unroll
  for (int m = 1; m < NM; ++m) {
    const double mq = (double)m * q;
    const double u2 = fma(d, u1, fma(-g, v1, mq * u0));
    const double v2 = fma(d, v1, fma(g, u1, mq * v0));
    u0 = u1;
    v0 = v1;
    u1 = u2;
    v1 = v2;
    A[m] = w * v1;
  }
}

// Order by cut (cuts of so many FWHM differ from line to line, in a block as much as over the
// list). A point at distance d from a block of kCutBlock lines takes those whose cut is at
// least d: with the block's lines in order of falling cut, its first so many. Their moments up
// to every 16th are kept as running sums, so a block costs a point one series and the lines
// around the boundary. A key holds the cut in units of cap / 4194303, rounded down, above
// the line's index in the block; the two bounds of a key's cut are a unit wider than that.
constexpr double kCutUnits = 4194303.0;
__host__ __device__ __forceinline__ uint32_t cut_key(double cut, double cap, int i) {
  return ((uint32_t)(cut / cap * kCutUnits) << 10) | (uint32_t)i;
}
__host__ __device__ __forceinline__ double cut_key_lower(uint32_t key, double unit) {
  return ((double)(key >> 10) - 1.0) * unit;
}
__host__ __device__ __forceinline__ double cut_key_upper(uint32_t key, double unit) {
  return ((double)(key >> 10) + 2.0) * unit;
}

#if defined(__HIPCC__)
// Exchange with the lane whose index differs by the mask 8, 7, 2 or 1 inside a row of 16
// lanes (row_ror:8, row_half_mirror, two quad permutations).
template <int kCtrl>
__device__ __forceinline__ double row_swap(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, 0xf, 0xf,
                                                            false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl,
                                                            0xf, 0xf, false);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
constexpr int kRowX8 = 0x128, kRowX7 = 0x141, kRowX2 = 0x4e, kRowX1 = 0xb1;

// One step of a halving sum: lanes with `up` keep the upper half of v[0 .. 2n), the others
// the lower, and add their partner's values of it.
template <int kCtrl, int n, int kV>
__device__ __forceinline__ void row_halve(double (&v)[kV], bool up) {
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const double x = v[i], y = v[i + n];
    const double give = up ? x : y, keep = up ? y : x;
    v[i] = keep + row_swap<kCtrl>(give);
  }
}

// One leaf from its 16 lanes' lines (lanes past the list's end repeat its last line with
// w = 0; the lines are in order, so the row's last lane holds the largest centre and Doppler
// width). Each lane forms the moments of its line; the sums over the row go by halving: at
// every step a lane keeps half of the values and adds its partner's, so 16 sums over 16 lanes
// take 15 exchanges, and lane i ends with moment i + 1 (28 moments: 2 i + 1 and 2 i + 2).
template <int NM, bool FW>
__device__ __forceinline__ void leaf_moments(double* nodes, int64_t leaf, double nu0, double w,
                                             double b, double g, double cut, int lane) {
  constexpr int kV = NM <= 16 ? 16 : 32;
  static_assert(NM <= 32 && kLeafLines == 16, "a leaf is a DPP row");
  const int row = lane & ~15, i = lane & 15;
  const double lo = __shfl(nu0, row), hi = __shfl(nu0, row + 15), bm = __shfl(b, row + 15);
  double gm = g;
  gm = fmax(gm, row_swap<kRowX8>(gm));
  gm = fmax(gm, row_swap<kRowX7>(gm));
  gm = fmax(gm, row_swap<kRowX2>(gm));
  gm = fmax(gm, row_swap<kRowX1>(gm));
  double cmin = cut, cmax = cut;
  if constexpr (FW) {
    cmin = fmin(cmin, row_swap<kRowX8>(cmin));
    cmax = fmax(cmax, row_swap<kRowX8>(cmax));
    cmin = fmin(cmin, row_swap<kRowX7>(cmin));
    cmax = fmax(cmax, row_swap<kRowX7>(cmax));
    cmin = fmin(cmin, row_swap<kRowX2>(cmin));
    cmax = fmax(cmax, row_swap<kRowX2>(cmax));
    cmin = fmin(cmin, row_swap<kRowX1>(cmin));
    cmax = fmax(cmax, row_swap<kRowX1>(cmax));
  }
  const double h = 0.5 * (hi - lo);
  const double s = sqrt(fma(h, h, gm * gm)) + far_beta<NM>() * bm;
  const double is = rcp64(s);
  double v[kV];
  {
    double A[NM];
    const double bs = b * is;
    line_moments<NM>(w, (nu0 - 0.5 * (lo + hi)) * is, g * is, 0.5 * bs * bs, A);
#pragma unroll
    for (int m = 0; m < kV; ++m) v[m] = m < NM ? A[m < NM ? m : 0] : 0.0;
  }
  row_halve<kRowX8, kV / 2>(v, (i & 8) != 0);
  row_halve<kRowX7, kV / 4>(v, (i & 4) != 0);
  row_halve<kRowX2, kV / 8>(v, (i & 2) != 0);
  row_halve<kRowX1, kV / 16>(v, (i & 1) != 0);
  constexpr int kPer = kV / 16;   // moments per lane
  const NodeRef<NM, double> nd{nodes + node_pos<NM>(leaf)};
#pragma unroll
  for (int m = 0; m < kPer; ++m)
    if (kPer * i + m < NM) nd.at(kNodeA + kPer * i + m) = v[m];
  if (i < kNodeA)
    nd.at(i) = i == kNodeLo ? lo : i == kNodeHi ? hi : i == kNodeS ? s : i == kNodeG ? gm
               : i == kNodeCutMin ? cmin : cmax;
}

// Moments of the wavefront's 64 lines (w = 0: none), for the FP64 path: lane i of every row
// of 16 ends with moments i + 1 (a) and i + 17 (b, 0 from moment 29 on). By halves, so that
// 16 values are held at a time.
__device__ __forceinline__ void wave_moments(double w, double d, double g, double q, int lane,
                                             double* a, double* b) {
  const int i = lane & 15;
  double u0 = 1.0, v0 = 0.0, u1 = d, v1 = g;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    double v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const int k = 16 * half + m + 1;   // moment k is w v1
      v[m] = k <= kMomFp64 ? w * v1 : 0.0;
      if (k < kMomFp64) {
        const double mq = (double)k * q;
        const double u2 = fma(d, u1, fma(-g, v1, mq * u0));
        const double v2 = fma(d, v1, fma(g, u1, mq * v0));
        u0 = u1;
        v0 = v1;
        u1 = u2;
        v1 = v2;
      }
    }
    row_halve<kRowX8, 8>(v, (i & 8) != 0);
    row_halve<kRowX7, 4>(v, (i & 4) != 0);
    row_halve<kRowX2, 2>(v, (i & 2) != 0);
    row_halve<kRowX1, 1>(v, (i & 1) != 0);
    double t = v[0];
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    *(half ? b : a) = t;
  }
}
// v of one lane (wave-uniform index), as a wave-uniform value
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// The largest v of the wavefront, wave-uniform.
__device__ __forceinline__ double wave_fmax(double v) {
  v = fmax(v, row_swap<kRowX8>(v));
  v = fmax(v, row_swap<kRowX7>(v));
  v = fmax(v, row_swap<kRowX2>(v));
  v = fmax(v, row_swap<kRowX1>(v));
  return fmax(fmax(lane_value(v, 0), lane_value(v, 16)),
              fmax(lane_value(v, 32), lane_value(v, 48)));
}
// One line at one point, with the cut test: the sums of the ragged ends of the far ranges
// (lines of a leaf that the cut of a point splits) and of the few leaves that are neither far
// nor inside the near range. FP32 path (NM = 16): the doubly shifted Lorentzian in FP64 where
// it holds to 5e-8 (r >= 74), else the tile kernel's forms; FP64 path: voigt_k64.
template <int NM>
__device__ __forceinline__ double one_line(double nu, double nu0, const LineRec& r) {
  const double d = nu - nu0;
  if (!(fabs(d) <= r.cut)) return 0.0;
  const double x = d * r.ib;
  if constexpr (NM == kMomFp32) {
    const double y2 = r.y * r.y;
    const double r2 = fma(x, x, y2);
    if (r2 >= 74.0 * 74.0)
      return kInvSqrtPi * r.sc * r.y * r2 * rcp64(fma(r2, r2 - 1.5, 2.0 * y2));
    if (r2 >= kT6R2)   // (y in FP64: K may lie below FP32's range)
      return kInvSqrtPi * r.sc * r.y * (double)asym_scaled<6>((float)y2, (float)r2);
    return r.sc * (double)voigt_k32(x, (float)r.y);
  } else {
    return r.sc * voigt_k64(x, r.y);
  }
}
#endif

}  // namespace xs
