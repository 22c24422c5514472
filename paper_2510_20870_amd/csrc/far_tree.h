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
// 5e-8 of every line's own contribution with 16 moments (theta 3.5, beta 2.3), and within
// 3e-14 with 28 (beta 2.6), measured against a reference Faddeeva routine over the whole
// range of h, g and b. All of it is FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_args.h"

namespace xs {

constexpr int kLeafLines = 64;       // one wavefront of lines
constexpr int kArity = 8;
constexpr double kFarTheta = 3.5;    // a group is far where |nu - c| >= kFarTheta * s
// moments of the FP32 and the FP64 path, and the weight of the Doppler width in s
constexpr int kMomFp32 = 16, kMomFp64 = 28;
constexpr double kBetaFp32 = 2.3, kBetaFp64 = 2.6;
template <int NM> constexpr double far_beta() { return NM == kMomFp32 ? kBetaFp32 : kBetaFp64; }

template <int NM>
struct alignas(16) FarNode {
  double lo, hi;   // centres of the group's first and last line
  double s;        // scale
  double g;        // largest Lorentz width
  double A[NM];    // A[m - 1]: moment m
};

// C(n, k) for n <= kMomFp64
struct BinomTable {
  double c[kMomFp64 + 1][kMomFp64 + 1];
};
constexpr BinomTable make_binom() {
  BinomTable t{};
  for (int n = 0; n <= kMomFp64; ++n) {
    t.c[n][0] = 1.0;
    for (int k = 1; k <= n; ++k)
      t.c[n][k] = t.c[n - 1][k - 1] + (k <= n - 1 ? t.c[n - 1][k] : 0.0);
  }
  return t;
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

// The series at X = nu - c: sum_m A_m s^m / X^(m+1).
template <int NM>
__host__ __device__ __forceinline__ double moment_sum(const double* A, double t, double rX) {
  double f = A[NM - 1];
#pragma unroll
  for (int m = NM - 2; m >= 0; --m) f = fma(f, t, A[m]);
  return f * t * rX;   // t = s / X, rX = 1 / X
}

#if defined(__HIPCC__)
// One leaf from its wavefront's lines (lanes past the list's end repeat its last line with
// w = 0; the lines are in order, so lane 63 holds the largest centre and Doppler width).
// Each lane forms the moments of its line; the sums over the wavefront go by halving: at
// every step a lane keeps half of the values and adds its partner's (NM + 1 exchanges
// instead of 6 NM), after which lane i holds the sum of one moment.
template <int NM>
__device__ __forceinline__ void leaf_moments(FarNode<NM>* node, double nu0, double w, double b,
                                             double g, int lane) {
  constexpr int kV = NM <= 16 ? 16 : 32;
  static_assert(NM <= 32, "moments of a wavefront reduction");
  const double lo = __shfl(nu0, 0), hi = __shfl(nu0, 63), bm = __shfl(b, 63);
  double gm = g;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) gm = fmax(gm, __shfl_xor(gm, o));
  const double h = 0.5 * (hi - lo);
  const double s = sqrt(fma(h, h, gm * gm)) + far_beta<NM>() * bm;
  const double is = 1.0 / s;
  double v[kV];
  {
    double A[NM];
    const double bs = b * is;
    line_moments<NM>(w, (nu0 - 0.5 * (lo + hi)) * is, g * is, 0.5 * bs * bs, A);
#pragma unroll
    for (int m = 0; m < kV; ++m) v[m] = m < NM ? A[m < NM ? m : 0] : 0.0;
  }
  int o = 32, m = 0;
#pragma unroll
  for (int n = kV / 2; n > 0; n >>= 1, o >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double give = up ? v[i] : v[i + n], keep = up ? v[i + n] : v[i];
      v[i] = keep + __shfl_xor(give, o);
    }
    m = 2 * m + (up ? 1 : 0);
  }
  double t = v[0];
#pragma unroll
  for (; o > 0; o >>= 1) t += __shfl_xor(t, o);
  constexpr int kRep = kWave / kV;   // lanes holding the same moment
  if ((lane & (kRep - 1)) == 0 && m < NM) node->A[m] = t;
  if (lane == 0) {
    node->lo = lo;
    node->hi = hi;
    node->s = s;
    node->g = gm;
  }
}
#endif

}  // namespace xs
