// Point kernel: the whole sum at a few neighbouring grid points by one wavefront, its lanes
// being lines (or line groups) instead of grid points.
//
// Section "Functionality of pyROX" (bullets "Compute line profiles", "Combine and save"). A
// wavefront takes kPointGroup neighbouring points of one (P, T) point. Around them it finds
// the lines that have to be summed one by one (the near range: leaves of the tree that are
// not far from every point), 64 lines at a time, one per lane, read once and evaluated at
// every point of the group; outside, up to the cut, the tree's nodes (far_tree.h), 64 at a
// time, one per lane; at the cut, the leaves that some points' cuts leave out, and the lines
// of the leaf that a cut splits. Each lane keeps one FP64 sum per point; they are added over
// the wavefront once, at the end.
//
// Why lanes are lines: with lanes as points of a tile, every line near the tile costs all 64
// lanes although its core covers a few points (3 to 60 of them on a 0.01 cm^-1 grid), its
// record passes through LDS, and its row classes and lane ranges have to be found first.
// Here a record is one coalesced load, no lane is idle for a point's sake, and whether a
// chunk of 64 neighbouring lines lies in the core or outside is nearly uniform. The group's
// width trades the loads and the tree walk, paid once per group, against the lines that only
// some of its points need. VALU-bound: about 55 instructions per 64 core pairs with y < 0.1,
// 30 outside the core. 20011 points of a list of 8700 lines/cm^-1 (0.3 bar, 435000 lines within
// the cut): 257 us at 66 % of the issue rate, 8.5 ms by the tile kernel over the whole window;
// FP64 path, 100003 points, 53000 lines within the cut: 300 us against 9.7 ms.
#include "far_tree.h"
#include "tile_kernel.h"

namespace xs {

constexpr int kEdgeQueue = 16;   // most leaves at the cut that go through the queue
constexpr int kPointRanges = 32;    // line ranges summed one by one, per wavefront
constexpr int kNodeList = 128;      // pending tree nodes, per wavefront

// Two searches at once, lanes 0-31 for one key and lanes 32-63 for the other: the first i in
// [lo, hi) with pred(a[i]), pred false and then true along the array (hi if none). The
// bounds are per half-wavefront.
template <class F>
__device__ __forceinline__ int pair_search(const double* __restrict__ a, int lo, int hi, F pred,
                                           int lane) {
  const int l5 = lane & 31, sh = lane & 32;
  while (__ballot(hi - lo > 32) != 0ull) {
    const int step = (hi - lo + 32) / 33;
    const int i = lo + (l5 + 1) * step;   // at most hi + 32 (step is rounded up)
    const bool before = i < hi && !pred(a[i]);
    const int c = __popc((uint32_t)(__ballot(before) >> sh));
    // the probes before the answer are the first c ones
    const int nlo = c > 0 ? lo + c * step + 1 : lo;
    hi = min(hi, lo + (c + 1) * step);
    lo = min(nlo, hi);
  }
  const int i = lo + l5;
  const bool before = i < hi && !pred(a[i]);
  return lo + __popc((uint32_t)(__ballot(before) >> sh));
}

// Sum of v over the wavefront for each of the R values, by halving (lane l holds value
// l / (64 / R) afterwards).
template <int R>
__device__ __forceinline__ double wave_sums(double (&v)[R], int lane) {
  int o = 32;
#pragma unroll
  for (int n = R / 2; n > 0; n >>= 1, o >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double x = v[i], y = v[i + n];
      const double give = up ? x : y, keep = up ? y : x;
      v[i] = keep + __shfl_xor(give, o);
    }
  }
  double t = v[0];
  for (; o > 0; o >>= 1) t += __shfl_xor(t, o);
  return t;
}

// The Dawson table of the small-y core in LDS, one 16-byte entry per node.
struct DawEntry {
  float F, F1, E, pad;
};

// voigt_core_small with its table in LDS.
__device__ __forceinline__ float core_small(const DawEntry* tab, double xd, float y) {
  const double ax = fabs(xd);
  const float kf = rintf(fminf((float)ax, 7.0f) * (float)kDawInvH);
  const DawEntry e = tab[(int)kf];
  const float x0 = kf * (float)(1.0 / kDawInvH);   // exact
  const float d = (float)(ax - (double)x0);
  const float m2x = -2.0f * x0;
  const float D0 = e.F, D1 = e.F1;
  const float D2 = fmaf(m2x, D1, -2.0f * D0);
  const float D3 = fmaf(m2x, D2, -4.0f * D1);
  const float D4 = fmaf(m2x, D3, -6.0f * D2);
  const float D5 = fmaf(m2x, D4, -8.0f * D3);
  const float D6 = fmaf(m2x, D5, -10.0f * D4);
  const float d2 = 0.5f * d, d3 = d * (1.0f / 3.0f), d4 = 0.25f * d;
  const float F1 = fmaf(d, fmaf(d2, fmaf(d3, fmaf(d4, D5, D4), D3), D2), D1);
  const float F3 = fmaf(d, fmaf(d2, fmaf(d3, D6, D5), D4), D3);
  const float F5 = fmaf(d, D6, D5);
  const float y2 = y * y;
  const float imF = y * fmaf(-y2 * (1.0f / 6.0f), fmaf(-y2 * 0.05f, F5, F3), F1);
  const float a = 2.0f * (x0 + d) * y;
  const float a2 = a * a;
  const float ca = fmaf(a2, fmaf(a2, fmaf(a2, -1.0f / 720.0f, 1.0f / 24.0f), -0.5f), 1.0f);
  const float g = e.E * exp32(fmaf(-fmaf(2.0f, x0, d), d, y2)) * ca;
  return fmaf(-2.0f * (float)kInvSqrtPi, imF, g);
}

// a b + c with c in a scalar register: one instruction (the compiler would copy the scalar
// pair into the accumulator first, two more per term of the loop below).
__device__ __forceinline__ double fma_s(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}

// Weideman's series (voigt_core64_n) for a wavefront of lines. The coefficients are real, so
// the sum follows from the recurrence b_n = a_n + 2 Re(Z) b_(n+1) - |Z|^2 b_(n+2) in real
// arithmetic, p = a_0 - |Z|^2 b_2 + Z b_1: two operations per term instead of four (|Z| < 1;
// within 15 % of Horner's rounding, which lies far below the truncation of these term counts).
template <int N>
__device__ __forceinline__ double core64(const double* a, double L, double x, double y) {
  const double lpy = L + y, lmy = L - y;
  const double x2 = x * x;
  const double iD = rcp64(fma(lpy, lpy, x2));
  const double zr = fma(lmy, lpy, -x2) * iD;
  const double t = zr + zr, u = -fma(lmy, lmy, x2) * iD;
  double b1 = fma_s(t, a[N - 1], a[N - 2]), b2 = a[N - 1];
#pragma unroll
  for (int n = N - 3; n >= 1; --n) {
    const double b = fma(t, b1, fma_s(u, b2, a[n]));   // (one step of the chain per term)
    b2 = b1;
    b1 = b;
  }
  // Re[2 p / (L - iz)^2 + 1 / (sqrt(pi) (L - iz))], Im p = 2 L x / D b_1
  const double pr = fma(u, b2, fma_s(zr, b1, a[0]));
  const double q = (4.0 * L) * x2 * lpy * iD;
  const double r = 2.0 * fma(pr, fma(lpy, lpy, -x2), -q * b1) * iD;
  return fma(lpy, kInvSqrtPi, r) * iD;
}

// The core form of a chunk of lines, one for the wavefront: none (every y >= 7: no point
// lies in the core), the FP32 small-y core (every y < 0.1), else the FP64 series with the
// term count that the chunk's smallest y needs (core_tier; 22 terms go with 24).
enum { kCoreNone, kCoreSmall, kCore16, kCore20, kCore24, kCoreAny };

// K(x, y) of one line per lane, FP32 path: the tile kernel's forms, outside the core the
// cheapest of three that serves every lane (the shifted Lorentzian within the launch's error
// budget eps, 3 terms from |z| = 20, 6 terms).
template <int CORE>
__device__ __forceinline__ double lane_k32(const DawEntry* tab, double x, double y, float y32,
                                           float y2, float eps) {
  const float xf = (float)x;
  const float r2 = fmaf(xf, xf, y2);
  const float c = (float)kInvSqrtPi * y32;
  if (__ballot(!(r2 >= kT3R2)) == 0ull) {
    if (__ballot(!shifted_lorentz_ok(y2, r2, eps)) == 0ull) return (double)(c * rcp32(r2 - 1.5f));
    return (double)(c * asym_scaled<3>(y2, r2));
  }
  float k = 0.0f;
  if constexpr (CORE == kCoreNone) {
    k = c * asym_scaled<6>(y2, r2);
  } else {
    const bool core = r2 < kT6R2;
    if (!core) k = c * asym_scaled<6>(y2, r2);
    if (core) {
      if constexpr (CORE == kCoreSmall) k = core_small(tab, x, y32);
      else if constexpr (CORE == kCore16) k = (float)core64<16>(kWeidA16, kWeidL16, x, y);
      else if constexpr (CORE == kCore20) k = (float)core64<20>(kWeidA20, kWeidL20, x, y);
      else if constexpr (CORE == kCore24) k = (float)core64<24>(kWeidA24, kWeidL24, x, y);
      else
        k = y32 < kTaylorY ? core_small(tab, x, y32)
                           : (float)voigt_core64_tier(core_tier(y), x, y);
    }
  }
  return (double)k;
}

// The same for lines of so small a y that the products above leave FP32's range (K falls below
// 1e-38 in the wing): y enters the wing's forms in FP64.
constexpr float kTinyY = 1e-20f;
__device__ __forceinline__ double lane_k32_tiny(const DawEntry* tab, double x, double y,
                                                float y32, float y2) {
  const float xf = (float)x;
  const float r2 = fmaf(xf, xf, y2);
  if (r2 >= kT6R2) return kInvSqrtPi * y * (double)asym_scaled<6>(y2, r2);
  return (double)(y32 < kTaylorY ? core_small(tab, x, y32)
                                 : (float)voigt_core64_tier(core_tier(y), x, y));
}

// The LDS of a workgroup, per wavefront but for the table.
template <int NM>
struct PointLds {
  DawEntry tab[NM == kMomFp32 ? kDawNodes : 1];
  int list[kWavesPerWG][kNodeList];
  int2 rng[kWavesPerWG][kPointRanges];
  int part[kWavesPerWG][2][kPointGroup];
  double cutl[kWavesPerWG][kPointGroup][2 * kLeafLines];
};

// The sums at the points [r0, r1) of the group from j0 (part s), true when they are stored. RUNS:
// where a gap between two of them holds many lines that are near neither (kGapLines), the
// run ends there: r1 is lowered, nothing is stored, and the caller asks again.
// FW: the lines' cuts differ (min(cap, mult FWHM)). The covered and the reachable lines then
// follow from bounds of the cut; between them lie leaves of which some lines reach a point and
// some do not.
template <int NM, bool FW, bool RUNS>
__device__ __forceinline__ bool point_run(const PointArgs& A, PointLds<NM>& lds, int lane, int wv,
                                          int64_t j0, int k, int s, int r0, int& r1) {
  constexpr int R = kPointGroup, NF = node_fields<NM>();
  auto& tab = lds.tab;
  auto& list = lds.list;
  auto& rng = lds.rng;
  auto& part = lds.part;
  auto& cutl = lds.cutl;
  const double v0 = A.grid[j0 + r0], v1 = A.grid[j0 + r1 - 1];
  const PtBounds pb = A.bounds[k];
  const double kb = pb.kb;
  const double cap = A.cut.cut;
  const int rec_n = A.rec_n;
  const double* nu = A.L.nu0 + A.rec_lo;
  const LineRec* recs = A.recs + (int64_t)k * rec_n;
  const double* nodes = A.nodes + (int64_t)k * A.dims.n_nodes * NF;
  auto node = [&](int l, int q) { return node_at<NM>(nodes, A.dims, l, (int64_t)q); };
  // the points: lane p (mod R) holds point p, read back as a wave-uniform value
  const uint64_t vb =
      __builtin_bit_cast(uint64_t, A.grid[j0 + min(max(lane & (R - 1), r0), r1 - 1)]);
  auto val = [&](int p) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)vb, p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(vb >> 32), p);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
  };

  double acc[R];
#pragma unroll
  for (int p = 0; p < R; ++p) acc[p] = 0.0;

  // ---- ranges. Per half-wavefront: lanes 0-31 the lines left of the points, 32-63 right.
  const bool right = lane >= 32;
  const int l5 = lane & 31;
  const double g_near = right ? v1 : v0;
  auto half = [&](int v, int side) { return __builtin_amdgcn_readlane(v, side * 32); };
  const double ulp = fabs(g_near) * 0x1p-48;
  // the largest cut of the lines on this side that can reach the points, and the smallest of
  // those (b_D grows with the centre, which is above zero also where a point is not)
  double cut_hi = cap, cut_lo = cap;
  if constexpr (FW) {
    cut_hi = cut_at(A.cut, pb.gmax, kb * (right ? v1 + cap : v1), true);
    cut_lo = cut_at(A.cut, pb.gmin, kb * fmax(right ? v0 : v0 - cut_hi, 0.0), false);
  }
  const bool one_cut = !FW || __ballot(cut_lo < cap) == 0ull;
  // reachable lines [e0, e1)
  const int end = pair_search(nu, 0, rec_n,
                              [&](double c) { return right ? c > v1 + cut_hi + ulp
                                                           : c >= v0 - cut_hi - ulp; }, lane);
  const int e0 = half(end, 0), e1 = half(end, 1);
  // lane kRep p holds point p's sum
  constexpr int kRep = kWave / R;
  auto put = [&](double t) {
    const int p = lane / kRep;
    if (lane % kRep != 0 || p < r0 || p >= r1) return;
    if (A.split > 1) {
      ((double*)A.out)[((int64_t)k * A.split + s) * A.n_grid + j0 + p] = t;
    } else {
      const int64_t o = (int64_t)(A.pt0 + k) * A.n_grid + j0 + p;
      if (A.out_f32) ((float*)A.out)[o] = (float)t;
      else ((double*)A.out)[o] = t;
    }
  };
  // No line in reach (a grid beyond its list's ends or in a gap of it). (24 (P, T) points of 1e5
  // points, 40 % of them past the list: 1.02 ms with the walks below, 0.97 so.)
  if (e0 >= e1) {
    put(0.0);
    return true;
  }
  // lines inside the cut of every point of the group, in leaves [c0, c1)
  const int cov = pair_search(nu, e0, e1,
                              [&](double c) { return right ? c - v0 > cut_lo : v1 - c <= cut_lo; },
                              lane);
  const int c0 = (half(cov, 0) + kLeafLines - 1) / kLeafLines, c1 = half(cov, 1) / kLeafLines;
  // near range, in leaves [a, b): first by the Doppler width, then grown over every leaf
  // that is not far
  const double reach = (kFarTheta * far_beta<NM>()) * kb * g_near;
  const int nr = pair_search(nu, e0, e1,
                             [&](double c) { return right ? c > v1 + reach : c >= v0 - reach; },
                             lane);
  if constexpr (RUNS) {
    // (4004 points in two bands 4000 cm^-1 apart, 1050 lines/cm^-1: 85 ms with the lines of the
    // gap summed at every point of one group, 0.24 so, 19.7 by tiles)
    const int n_near = half(nr, 1) - half(nr, 0);
    const double wide = 2.0 * kFarTheta * (pb.gmax + far_beta<NM>() * kb * fabs(v1));
    if (n_near > kGapLines && v1 - v0 > wide) {
      const double per = (double)n_near / (v1 - v0);   // lines per wavenumber, rather too many
      for (int p = r0 + 1; p < r1; ++p) {
        const double gap = val(p) - val(p - 1);
        const int most = gap > 0.5 * (v1 - v0) ? kGapLines : kStepLines;
        if ((gap - wide) * per > (double)most) {
          r1 = p;
          return false;
        }
      }
    }
  }
  int a = half(nr, 0) / kLeafLines, b = (half(nr, 1) + kLeafLines - 1) / kLeafLines;
  // distance of a node outwards from the nearest point
  auto is_far = [&](const NodeRef<NM, const double>& f) {
    const double c = f.c();
    return (right ? c - v1 : v0 - c) >= kFarTheta * f.s();
  };
  auto grow = [&](int l, int& lo, int& hi, int from, int to) {
    for (;;) {
      const int q = right ? hi + l5 : lo - 1 - l5;
      bool bad = false;
      if (right ? q < to : q >= from) bad = !is_far(node(l, q));
      const uint64_t m = __ballot(bad);
      if (m == 0ull) break;
      const uint32_t ml = (uint32_t)m, mr = (uint32_t)(m >> 32);
      lo -= ml ? 32 - __clz((int)ml) : 0;
      hi += mr ? 32 - __clz((int)mr) : 0;
      // (the rest of the 32 are far; a node beyond that is not is found when it is taken)
      if (((ml | mr) >> 16) == 0u) break;
    }
  };
  grow(0, a, b, c0, c1);

  int n_rng = 1;
  bool mask = a < c0 || b > c1;   // the near range holds lines outside some point's cut
  const int n0 = max(e0, min(a * kLeafLines, rec_n)), n1 = min(e1, min(b * kLeafLines, rec_n));
  if (lane == 0) rng[wv][0] = make_int2(n0, max(n0, n1));
  if (lane < 2 * R) part[wv][lane >= R][lane & (R - 1)] = -1;
  wave_sync();

  // ---- tree nodes inside every point's cut, 64 at a time: one per lane
  bool whole = false;   // too many nodes that are not far: sum every line of the window
  int n_list = 0, round = 0;
  // adds the lane's moments (use: it has some) about c, scale sc, to every point's sum; lanes
  // without take zeros about a centre beyond the last point (which may be below zero)
  auto add_moments = [&](double c, double sc, bool use, auto moment) {
    const double cc = use ? c : v1 + fabs(v1) + 1.0;
    double M[NM];
#pragma unroll
    for (int t = 0; t < NM; ++t) M[t] = use ? moment(t) : 0.0;
#pragma unroll
    for (int p = 0; p < R; ++p) {
      const double rX = rcp64(val(p) - cc), t = sc * rX;
      double h = M[NM - 1];
#pragma unroll
      for (int m2 = NM - 2; m2 >= 0; --m2) h = fma(h, t, M[m2]);
      acc[p] = fma(h * t, rX, acc[p]);
    }
  };
  // lanes with `bad`: node (l, q) is summed line by line
  auto to_ranges = [&](bool bad, int l, int q) {
    const uint64_t m = __ballot(bad);
    if (m == 0ull) return;
    const int add = __popcll(m);
    if (n_rng + add > kPointRanges) {
      whole = true;
      return;
    }
    const int i0 = q << (kArityBits * l), i1 = (q + 1) << (kArityBits * l);
    if (bad)
      rng[wv][n_rng + __popcll(m & ((1ull << lane) - 1ull))] =
          make_int2(i0 * kLeafLines, min(i1 * kLeafLines, rec_n));
    n_rng += add;
  };
  auto flush = [&](int n) {
    wave_sync();
    const int id = lane < n ? list[wv][lane] : -1;
    const int l = id >> 27, q = id & 0x7ffffff;
    const bool in = id >= 0;
    NodeRef<NM, const double> f{nodes};
    if (in) f = node(l, q);
    const double c = f.c(), sc = f.s();
    const bool bad = in && !(fmax(v0 - c, c - v1) >= kFarTheta * sc);
    to_ranges(bad, l, q);
    if (round++ % A.split == s)
      add_moments(c, sc, in && !bad, [&](int t) { return f.at(kNodeA + t); });
    // the nodes not taken yet move to the front
    const int rest = lane + kWave < n_list ? list[wv][kWave + lane] : 0;
    wave_sync();
    list[wv][lane] = rest;
    n_list -= n;
    wave_sync();
  };
  {
    int al = a, bl = b, lo = c0, hi = c1;   // near and covered ranges in nodes of level l
    bool on_l = al > lo, on_r = bl < hi;
    for (int l = 0; (on_l || on_r) && l < A.dims.levels; ++l) {
      // the next level's ranges: the near range out to whole parents that are not far, the
      // covered range in to whole parents
      int pa = al >> kArityBits, pb = (bl + kArity - 1) >> kArityBits;
      const int plo = (lo + kArity - 1) >> kArityBits, phi = hi >> kArityBits;
      bool up_l = false, up_r = false;
      if (l + 1 < A.dims.levels) {
        grow(l + 1, pa, pb, on_l ? plo : 0x7fffffff, on_r ? phi : -1);
        up_l = on_l && pa > plo;
        up_r = on_r && pb < phi;
      }
      // left: [lo, plo) and [pa, al) in children where parents go on, else [lo, al)
      const int s0 = on_l ? (up_l ? (plo << kArityBits) - lo : al - lo) : 0;
      const int s1 = up_l ? al - (pa << kArityBits) : 0;
      const int s2 = on_r ? (up_r ? (pb << kArityBits) - bl : hi - bl) : 0;
      const int s3 = up_r ? hi - (phi << kArityBits) : 0;
      const int n4 = s0 + s1 + s2 + s3;
      for (int o = 0; o < n4; o += kWave) {
        const int i = o + lane;
        if (i < n4) {
          const int q = i < s0 ? lo + i
                        : i < s0 + s1 ? (pa << kArityBits) + (i - s0)
                        : i < s0 + s1 + s2 ? bl + (i - s0 - s1)
                                           : (phi << kArityBits) + (i - s0 - s1 - s2);
          list[wv][n_list + lane] = (l << 27) | q;
        }
        n_list += min(kWave, n4 - o);
        if (n_list >= kWave) flush(kWave);
      }
      al = pa;
      bl = pb;
      lo = plo;
      hi = phi;
      on_l = up_l;
      on_r = up_r;
    }
    if (n_list > 0) flush(n_list);
  }

  // ---- leaves at the cut: left [e0 / 16, min(a, c0)), right [max(b, c1), e1 / 16 up)
  const int la = e0 / kLeafLines, lb = min(a, c0);
  const int ra = max(b, c1), rb = (e1 + kLeafLines - 1) / kLeafLines;
  const int nl = max(lb - la, 0), n_edge = nl + max(rb - ra, 0);
  auto edge_leaf = [&](int i) { return i < nl ? la + i : ra + (i - nl); };
  // One cut and more than kEdgeQueue leaves (a dense list): a leaf counts for the points whose
  // cut holds all of it, and the leaf that a cut splits is noted. Few leaves, or different
  // cuts: below, line by line where a leaf is not inside every cut. (The
  // queue sums a leaf's 16 lines at every point, 64 leaves by their moments cost one node per
  // lane and the lines of the two split leaves. A 250 cm^-1 window of 8696 lines/cm^-1 takes
  // 257 us by leaf and 302 us with the queue.)
  const bool by_leaf = one_cut && n_edge > kEdgeQueue;
  if (by_leaf) {
    const double cut = cap;
    for (int o = 0; o < n_edge; o += kWave) {
      const int i = o + lane;
      const bool in = i < n_edge;
      const int q = in ? edge_leaf(i) : 0;
      const NodeRef<NM, const double> f = node(0, q);
      const double lo = f.lo(), hi = f.hi(), c = f.c(), sc = f.s();
      const bool bad = in && !(fmax(v0 - c, c - v1) >= kFarTheta * sc);
      if (__ballot(bad) != 0ull) {
        mask = true;
        to_ranges(bad, 0, q);
      }
      const bool mine = round++ % A.split == s;
      const bool use = in && !bad && mine;
      double M[NM];
#pragma unroll
      for (int t = 0; t < NM; ++t) M[t] = use ? f.at(kNodeA + t) : 0.0;
#pragma unroll
      for (int p = 0; p < R; ++p) {
        const double v = val(p);
        const bool lo_in = fabs(v - lo) <= cut, hi_in = fabs(v - hi) <= cut;
        if (in && !bad && lo_in != hi_in) part[wv][i >= nl][p] = q;
        const double rX = rcp64(v - c), t = sc * rX;
        double h = M[NM - 1];
#pragma unroll
        for (int m2 = NM - 2; m2 >= 0; --m2) h = fma(h, t, M[m2]);
        if (use && lo_in && hi_in) acc[p] = fma(h * t, rX, acc[p]);
      }
    }
    wave_sync();
  }
  // Few leaves or different cuts: the lines that reach some point are gathered in a queue and
  // summed 64 at a time, one per lane.
  int turn = 0;   // the part that takes the next chunk
  auto my_turn = [&]() {
    const bool mine = turn == s;
    turn = turn + 1 == A.split ? 0 : turn + 1;
    return mine;
  };
  if (!by_leaf && !whole) {
    int n_q = 0;
    auto sum_queue = [&](int n) {
      wave_sync();
      const bool ok = lane < n;
      const int i = list[wv][ok ? lane : 0];
      const int rest = lane + kWave < n_q ? list[wv][kWave + lane] : 0;
      wave_sync();
      list[wv][lane] = rest;
      n_q -= n;
      wave_sync();
      if (!my_turn()) return;
      const double c = nu[i];
      const LineRec lr = recs[i];
      // the shifted or the doubly shifted Lorentzian within the error budget at both ends
      // of the group, else the six-term series (x and r^2 in FP64, the reciprocals in
      // FP32); FP64 path: voigt_k64, which is outside its core here
      const double w = ok ? lr.sc : 0.0, y2 = lr.y * lr.y;
      auto far_points = [&](double w1, double add, auto k_of) {
#pragma unroll
        for (int p = 0; p < R; ++p) {
          const double d = val(p) - c, x = d * lr.ib;
          const double wp = fabs(d) <= lr.cut ? w1 : 0.0;
          acc[p] = fma(k_of(fma(x, x, add)), wp, acc[p]);
        }
      };
      if constexpr (NM == kMomFp32) {
        const double xa = (v0 - c) * lr.ib, xb = (v1 - c) * lr.ib;
        const float y2f = (float)y2, rn = (float)(fmin(xa * xa, xb * xb) + y2);
        const double w1 = w * lr.y * kInvSqrtPi;
        if (__ballot(!shifted_lorentz_ok(y2f, rn, A.l1_eps)) == 0ull)
          far_points(w1, y2 - 1.5, [&](double r) { return (double)rcp32((float)r); });
        else if (__ballot(!dshift_ok(rn, A.l1_eps)) == 0ull)
          far_points(w1, y2, [&](double r2) {
            const float r = (float)r2;
            return (double)rcp32(fmaf(2.0f * y2f, rcp32(r), r - 1.5f));
          });
        else
          far_points(w1, y2,
                     [&](double r2) { return (double)asym_scaled<6>(y2f, (float)r2); });
      } else {
        far_points(w, y2, [&](double r2) {
          return r2 >= kFarR2_64 ? voigt_far64(r2, lr.y) : voigt_mid64(r2, lr.y);
        });
      }
    };
    // The leaves one round of 64 after the other; first, where the lines' cuts differ, the
    // whole blocks of kCutBlock lines that are far and ordered by cut, 64 at a time. (A block
    // that is not far goes leaf by leaf.)
    const int lx = max(la, lb), ry = max(ra, rb);
    int x0 = lx, x1 = lx, y0 = ry, y1 = ry;   // left and right whole blocks, in leaves
    constexpr int kPer = kCutBlock / kLeafLines;
    if constexpr (FW) {
      const int p0 = (la + kPer - 1) / kPer * kPer, p1 = min(lb / kPer, A.order.blocks) * kPer;
      if (p0 < p1) x0 = p0, x1 = p1;
      const int q0 = (ra + kPer - 1) / kPer * kPer, q1 = min(rb / kPer, A.order.blocks) * kPer;
      if (q0 < q1) y0 = q0, y1 = q1;
    }
    const int nx = (x1 - x0) / kPer, n_blk = A.order.blocks ? nx + (y1 - y0) / kPer : 0;
    const int n_leaf = n_blk ? n_edge - n_blk * kPer : n_edge;
    auto edge_rest = [&](int i) {   // leaf i of those outside the blocks
      if (!FW || n_blk == 0) return edge_leaf(i);
      if (i < x0 - la) return la + i;
      i -= x0 - la;
      if (i < lx - x1) return x1 + i;
      i -= lx - x1;
      return i < y0 - ra ? ra + i : y1 + (i - (y0 - ra));
    };
    const uint32_t* keys = A.order.keys + (int64_t)k * A.order.blocks * kCutBlock;
    const double* pre = A.order.pre + (int64_t)k * A.order.blocks * (kPer * NM);
    const double unit = cap * (1.0 / kCutUnits);
    int blk = 0;            // the lane's block of the last round of blocks
    uint64_t todo = 0ull;   // lanes whose block is still to go leaf by leaf
    for (int o_blk = 0, o_leaf = 0;;) {
      // per lane: groups [ent, ent + cnt) of 16 lines whose lines are tested one by one
      int ent = 0, cnt = 0;
      bool sorted = false;
      if (FW && todo == 0ull && o_blk < n_blk) {
        const int e = o_blk + lane;
        o_blk += kWave;
        const bool in = e < n_blk, is_left = e < nx;
        blk = !in ? 0 : is_left ? x0 / kPer + e : y0 / kPer + (e - nx);
        const NodeRef<NM, const double> f = node(kCutLevel, blk);
        const double lo = f.lo(), hi = f.hi(), c = f.c(), sc = f.s();
        const bool far = fmax(v0 - c, c - v1) >= kFarTheta * sc;
        todo = __ballot(in && !far);
        const double dmin = is_left ? v0 - hi : lo - v1, dmax = is_left ? v1 - lo : hi - v0;
        // groups inside every point's cut, and groups that reach some point
        const uint32_t* kb_ = keys + (int64_t)blk * kCutBlock;
        int n_in = 0, n_reach = 0;
        if (in && far) {
#pragma unroll
          for (int st = kPer; st >= 1; st /= 2) {
            if (n_in + st <= kPer &&
                cut_key_lower(kb_[(n_in + st) * kLeafLines - 1], unit) >= dmax)
              n_in += st;
            if (n_reach + st <= kPer &&
                cut_key_upper(kb_[(n_reach + st - 1) * kLeafLines], unit) >= dmin)
              n_reach += st;
          }
          ent = blk * kPer + n_in;
          cnt = max(n_reach - n_in, 0);
        }
        sorted = true;
        if (__ballot(n_in > 0) != 0ull && round++ % A.split == s) {
          const double* row = pre + ((int64_t)blk * kPer + max(n_in - 1, 0)) * NM;
          add_moments(c, sc, n_in > 0, [&](int t) { return row[t]; });
        }
      } else {
        bool in = true, is_left;
        int leaf;
        if (FW && todo != 0ull) {
          const int id = __builtin_amdgcn_readlane(blk, __builtin_ctzll(todo));
          todo &= todo - 1ull;
          leaf = id * kPer + lane;
          is_left = leaf < lx;
        } else if (o_leaf < n_leaf) {
          const int e = o_leaf + lane;
          o_leaf += kWave;
          in = e < n_leaf;
          leaf = in ? edge_rest(e) : 0;
          is_left = leaf < lx;
        } else {
          break;
        }
        const NodeRef<NM, const double> f = node(0, leaf);
        const double lo = f.lo(), hi = f.hi(), c = f.c(), sc = f.s();
        const double cmax = FW ? f.at(kNodeCutMax) : cap, cmin = FW ? f.at(kNodeCutMin) : cap;
        const bool out = !in || (is_left ? v0 - hi : lo - v1) > cmax;
        const bool far = fmax(v0 - c, c - v1) >= kFarTheta * sc;
        // inside every line's cut at every point: by its moments
        const bool all = !out && far && (is_left ? v1 - lo : hi - v0) <= cmin;
        if (__ballot(all) != 0ull && round++ % A.split == s)
          add_moments(c, sc, all, [&](int t) { return f.at(kNodeA + t); });
        const bool near = !out && !far;
        if (__ballot(near) != 0ull) {
          mask = true;
          to_ranges(near, 0, leaf);
        }
        ent = leaf;
        cnt = !out && far && !all ? 1 : 0;
      }
      // four groups at a time, one per row of 16 lanes
      uint64_t m4 = __ballot(cnt > 0);
      while (m4 != 0ull) {
        int q = -1;
#pragma unroll
        for (int t = 0; t < kWave / kLeafLines; ++t) {
          if (m4 != 0ull) {
            const int src = __builtin_ctzll(m4);
            const int id = __builtin_amdgcn_readlane(ent, src);
            if (__builtin_amdgcn_readlane(cnt, src) == 1) m4 &= m4 - 1ull;
            if (lane == src) {
              ++ent;
              --cnt;
            }
            if (lane / kLeafLines == t) q = id;
          }
        }
        int i = q * kLeafLines + (lane & (kLeafLines - 1));
        if (FW && sorted && q >= 0) i = (i & -kCutBlock) | (int)(keys[i] & (kCutBlock - 1));
        bool take = false;
        if (q >= 0 && i < rec_n) {
          const double ci = nu[i];
          const double ct = FW ? recs[i].cut : cap;
          take = fabs(v0 - ci) <= ct || fabs(v1 - ci) <= ct;
        }
        const uint64_t m = __ballot(take);
        if (take) list[wv][n_q + __popcll(m & ((1ull << lane) - 1ull))] = i;
        n_q += __popcll(m);
        if (n_q >= kWave) sum_queue(kWave);
      }
    }
    if (n_q > 0) sum_queue(n_q);
  }
  if (whole) {
    // (the same decision in every part of the group)
#pragma unroll
    for (int p = 0; p < R; ++p) acc[p] = 0.0;
    mask = true;
    n_rng = 1;
    if (lane == 0) rng[wv][0] = make_int2(e0, e1);
  } else if (by_leaf && s == 0) {
    // the split leaves: lanes 0-15 the left one's lines, 16-31 the right one's, per point
    // (through LDS, so that the sums keep their registers in a loop that is not unrolled)
#pragma unroll 1
    for (int p = 0; p < R; ++p) {
      const int q = lane < 2 * kLeafLines ? part[wv][lane >= kLeafLines][p] : -1;
      const int i = q * kLeafLines + (lane & (kLeafLines - 1));
      double t = 0.0;
      if (q >= 0 && i < rec_n) t = one_line<NM>(val(p), nu[i], recs[i]);
      if (lane < 2 * kLeafLines) cutl[wv][p][lane] = t;
    }
    wave_sync();
#pragma unroll
    for (int p = 0; p < R; ++p)
      if (lane < 2 * kLeafLines) acc[p] += cutl[wv][p][lane];
  }
  wave_sync();

  // ---- lines of the ranges, 64 at a time: one per lane
  for (int r = 0; r < n_rng; ++r) {
    // (the walk's state in scalar registers)
    const int first = __builtin_amdgcn_readfirstlane(rng[wv][r].x);
    const int last = __builtin_amdgcn_readfirstlane(rng[wv][r].y) - 1;
    for (int base = first; base <= last; base += kWave) {
      if (!my_turn()) continue;
      const int i = min(base + lane, last);
      const double c = nu[i];
      const LineRec lr = recs[i];
      const double sc = base + lane <= last ? lr.sc : 0.0;
      // adds the line to every point's sum with the given K
      auto points = [&](auto k_of) {
#pragma unroll
        for (int p = 0; p < R; ++p) {
          const double d = val(p) - c;
          const double kk = k_of(d * lr.ib);
          double w = sc;
          if (mask) w = fabs(d) <= lr.cut ? sc : 0.0;
          acc[p] = fma(w, kk, acc[p]);
        }
      };
      if constexpr (NM == kMomFp32) {
        const float y32 = (float)lr.y, y2 = y32 * y32;
        auto all = [&](bool t) { return __ballot(!t) == 0ull; };
        auto with = [&](auto core) {
          points([&](double x) {
            return lane_k32<decltype(core)::value>(tab, x, lr.y, y32, y2, A.l1_eps);
          });
        };
        if (!all(y32 >= kTinyY))
          points([&](double x) { return lane_k32_tiny(tab, x, lr.y, y32, y2); });
        else if (all(y2 >= kT6R2)) with(std::integral_constant<int, kCoreNone>{});
        else if (all(y32 < kTaylorY)) with(std::integral_constant<int, kCoreSmall>{});
        else if (all(lr.y >= 1.0)) with(std::integral_constant<int, kCore16>{});
        else if (all(lr.y >= 0.3)) with(std::integral_constant<int, kCore20>{});
        else if (all(lr.y >= 0.01)) with(std::integral_constant<int, kCore24>{});
        else with(std::integral_constant<int, kCoreAny>{});
      } else {
        points([&](double x) { return voigt_k64(x, lr.y); });
      }
    }
  }

  put(wave_sums<R>(acc, lane));
  return true;
}

// RUNS: grids with gaps of many lines (a variant of its own, as the loop costs the others spills
// and 9 % of their time).
template <int NM, bool FW, bool RUNS>
__global__ __launch_bounds__(kBlock, 4) void xs_point_kernel(PointArgs A) {
  constexpr int R = kPointGroup;
  __shared__ PointLds<NM> lds;
  if constexpr (NM == kMomFp32) {
    for (int t = threadIdx.x; t < kDawNodes; t += blockDim.x)
      lds.tab[t] = {kDawF[t], kDawF1[t], kDawE[t], 0.0f};
    __syncthreads();
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = logical_wg() * kWavesPerWG + wv;
  if (item >= A.n_groups * A.n_pt * A.split) return;
  // parts of a group and neighbouring groups of one (P, T) point lie next to each other
  const int s = (int)(item % A.split);
  const int64_t gi = item / A.split;
  const int k = (int)(gi / A.n_groups);
  const int64_t j0 = (A.g0 + gi % A.n_groups) * R;
  const int jn = (int)min((int64_t)R, A.n_grid - j0);
  int r1 = jn;
  if constexpr (!RUNS) {
    point_run<NM, FW, false>(A, lds, lane, wv, j0, k, s, 0, r1);
  } else {
    for (int r0 = 0; r0 < jn;)
      if (point_run<NM, FW, true>(A, lds, lane, wv, j0, k, s, r0, r1)) {
        r0 = r1;
        r1 = jn;
      }
  }
}

template <int NM, bool FW>
static void launch_point_as(const PointArgs& A, dim3 grid, dim3 block, hipStream_t st) {
  if (A.runs) hipLaunchKernelGGL((xs_point_kernel<NM, FW, true>), grid, block, 0, st, A);
  else hipLaunchKernelGGL((xs_point_kernel<NM, FW, false>), grid, block, 0, st, A);
}

hipError_t launch_point(const PointArgs& A, int moments, hipStream_t st) {
  const int64_t items = A.n_groups * A.n_pt * A.split;
  if (items <= 0) return hipSuccess;
  const dim3 grid = wg_grid(phys_workgroups((items + kWavesPerWG - 1) / kWavesPerWG)),
             block(kBlock);
  const bool fw = A.cut.kind != kCutFixed;
  if (moments == kMomFp32 && fw) launch_point_as<kMomFp32, true>(A, grid, block, st);
  else if (moments == kMomFp32) launch_point_as<kMomFp32, false>(A, grid, block, st);
  else if (fw) launch_point_as<kMomFp64, true>(A, grid, block, st);
  else launch_point_as<kMomFp64, false>(A, grid, block, st);
  return hipGetLastError();
}

}  // namespace xs
