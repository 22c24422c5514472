// Far field by moments of line groups (far_tree.h): the levels of the tree above its leaves,
// and the far kernel, which sums for every grid tile the lines outside its near range.
//
// Section "Functionality of pyROX" (bullets "Compute line profiles", "Combine and save"): the
// sum over every line inside the cutoff; here the lines far from a grid point enter group by
// group, with the same cutoff test per (line, point) pair.
#include "far_tree.h"
#include "tile_kernel.h"

namespace xs {

static __device__ const BinomTable kBinom = make_binom();

// Scale of a node from its extent and its largest Lorentz width (b = kb nu0).
template <int NM>
__device__ __forceinline__ double node_scale(double lo, double hi, double g, double kb) {
  const double h = 0.5 * (hi - lo);
  return sqrt(fma(h, h, g * g)) + far_beta<NM>() * (kb * hi);
}

// Moment m of a parent (centre c, 1/scale is) from n children.
template <int NM>
__device__ __forceinline__ double shift_moment(const FarNode<NM>* ch, int n, int m, double c,
                                               double is) {
  double sum = 0.0;
  for (int q = 0; q < n; ++q) {
    const FarNode<NM>& f = ch[q];
    const double D = (0.5 * (f.lo + f.hi) - c) * is, R = f.s * is;
    // sum_j C(m, j) D^j R^(m-j) A_(m-j), Horner in D
    double pw = R;
    double acc = kBinom.c[m][m - 1] * pw * f.A[0];
    for (int j = m - 2; j >= 0; --j) {
      pw *= R;
      acc = fma(acc, D, kBinom.c[m][j] * pw * f.A[m - j - 1]);
    }
    sum += acc;
  }
  return sum;
}

// Two levels at once: a workgroup takes kArity^2 nodes of level l (staged in LDS), writes
// their kArity parents and, where the level exists, the one parent of those. One thread per
// (parent, moment).
template <int NM>
__global__ __launch_bounds__(256) void xs_tree_up_kernel(ParamArgs A, int l) {
  constexpr int kChild = kArity * kArity;
  __shared__ FarNode<NM> ch[kChild], up[kArity];
  const int k = blockIdx.y;
  FarNode<NM>* nodes = (FarNode<NM>*)A.nodes + (int64_t)k * A.dims.n_nodes;
  const double kb =
      make_pt(A.sp, A.pts[2 * (A.pt0 + k)], A.pts[2 * (A.pt0 + k) + 1]).dopp / kCLight;
  const int64_t c0 = (int64_t)blockIdx.x * kChild;
  const int nc = (int)min((int64_t)kChild, A.dims.cnt[l] - c0);
  constexpr int kWords = sizeof(FarNode<NM>) / sizeof(double);
  typedef double __attribute__((may_alias)) word;
  {
    const word* src = (const word*)(nodes + A.dims.off[l] + c0);
    word* dst = (word*)ch;
    for (int t = threadIdx.x; t < nc * kWords; t += blockDim.x) dst[t] = src[t];
  }
  __syncthreads();
  auto level = [&](const FarNode<NM>* from, int nfrom, FarNode<NM>* lds, FarNode<NM>* to) {
    const int np = (nfrom + kArity - 1) / kArity;
    for (int t = threadIdx.x; t < np * NM; t += blockDim.x) {
      const int q = t / NM, m = t - q * NM + 1;
      const FarNode<NM>* f = from + q * kArity;
      const int n = min(kArity, nfrom - q * kArity);
      const double lo = f[0].lo, hi = f[n - 1].hi;
      double g = 0.0;
      for (int i = 0; i < n; ++i) g = fmax(g, f[i].g);
      const double s = node_scale<NM>(lo, hi, g, kb);
      const double a = shift_moment<NM>(f, n, m, 0.5 * (lo + hi), 1.0 / s);
      to[q].A[m - 1] = a;
      if (lds) lds[q].A[m - 1] = a;
      if (m == 1) {
        to[q].lo = lo;
        to[q].hi = hi;
        to[q].s = s;
        to[q].g = g;
        if (lds) {
          lds[q].lo = lo;
          lds[q].hi = hi;
          lds[q].s = s;
          lds[q].g = g;
        }
      }
    }
    return np;
  };
  const bool two = l + 2 < A.dims.levels;
  const int np = level(ch, nc, two ? up : nullptr,
                       nodes + A.dims.off[l + 1] + (int64_t)blockIdx.x * kArity);
  if (!two) return;
  __syncthreads();
  level(up, np, nullptr, nodes + A.dims.off[l + 2] + blockIdx.x);
}

hipError_t launch_tree_up(const ParamArgs& A, hipStream_t st) {
  if (A.n <= 0 || A.n_pt <= 0) return hipSuccess;
  for (int l = 0; l + 1 < A.dims.levels; l += 2) {
    const int64_t blocks = (A.dims.cnt[l] + kArity * kArity - 1) / (kArity * kArity);
    const dim3 grid((unsigned)blocks, (unsigned)A.n_pt), block(256);
    if (A.moments == kMomFp32)
      hipLaunchKernelGGL(xs_tree_up_kernel<kMomFp32>, grid, block, 0, st, A, l);
    else
      hipLaunchKernelGGL(xs_tree_up_kernel<kMomFp64>, grid, block, 0, st, A, l);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
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
    return r.sc * (double)voigt_k32(x, (float)r.y);
  } else {
    return r.sc * voigt_k64(x, r.y);
  }
}

// Far kernel. One workgroup per (tile, P-T point): wavefronts 0 and 1 take the groups left
// and right of the near range that are inside the cut of every point of the tile (the same
// nodes for all lanes), wavefronts 2 and 3 the lines beyond, up to each point's own cut
// (a walk over nodes per lane). What bounds it is the latency of a node's loads and of its
// Horner chain: the node counts grow with the logarithm of the window, not with its lines.
//
// Near range: from the tile outwards, the leaves up to the last of the leaves nearby that are
// not far from the whole tile (|nu - c| < theta s for some point); each 64-leaf group is
// tested at once, and the range ends at the first group of far leaves.
template <int NM>
__global__ __launch_bounds__(kBlock) void xs_far_kernel(FarArgs A) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = xcd_logical_wg(blockIdx.x);
  if (item >= A.n_items) return;   // the whole workgroup
  const int k = (int)(item % A.n_pt);
  const int64_t tile = A.tile_order ? (int64_t)A.tile_order[item / A.n_pt] : item / A.n_pt;
  const int64_t j0 = tile * kWave * A.P;
  const int64_t jl = min(j0 + (int64_t)kWave * A.P, A.n_grid) - 1;
  const double g0 = A.grid[j0], g1 = A.grid[jl];
  const int pt = A.pt0 + k;
  const double kb = make_pt(A.sp, A.pts[2 * pt], A.pts[2 * pt + 1]).dopp / kCLight;
  const double cut = A.cut;
  const double* nu = A.L.nu0 + A.rec_lo;
  const LineRec* recs = A.recs + (int64_t)k * A.rec_n;
  const FarNode<NM>* nodes = (const FarNode<NM>*)A.nodes + (int64_t)k * A.dims.n_nodes;
  const int levels = A.dims.levels;
  const bool left = (wv & 1) == 0, edge = wv >= 2;
  auto node_at = [&](int l, int64_t q) -> const FarNode<NM>& {
    return nodes[A.dims.off[l] + q];
  };
  // signed distance from v outwards to the node's centre
  auto dist = [&](const FarNode<NM>& f, double v) {
    const double c = 0.5 * (f.lo + f.hi);
    return left ? v - c : c - v;
  };
  const double g_near = left ? g0 : g1;   // the tile's point nearest to this side's lines

  // this side's ranges, in lines of the record range: near boundary (a leaf boundary),
  // lines inside the cut of every point up to `cov` (leaf boundary), reachable up to `end`
  int64_t near_b, cov, end;   // near_b, cov: leaf indices
  const double reach = (kFarTheta * far_beta<NM>()) * kb * g_near;
  if (left) {
    near_b = wave_search<false>(nu, A.rec_n, g0 - reach, lane) / kLeafLines;
    end = wave_search<false>(nu, A.rec_n, g0 - cut - fabs(g0) * 0x1p-48, lane);
    const int64_t c = end + wave_search_pred(nu + end, A.rec_n - end,
                                             [&](double v) { return g1 - v <= cut; }, lane);
    cov = (c + kLeafLines - 1) / kLeafLines;
  } else {
    near_b = (wave_search<true>(nu, A.rec_n, g1 + reach, lane) + kLeafLines - 1) / kLeafLines;
    end = wave_search<true>(nu, A.rec_n, g1 + cut + fabs(g1) * 0x1p-48, lane);
    cov = wave_search_pred(nu, end, [&](double v) { return v - g0 > cut; }, lane) / kLeafLines;
  }
  // grow the near range over leaves that are not far from the tile
  for (;;) {
    const int64_t q = left ? near_b - 1 - lane : near_b + lane;
    const bool in = left ? q >= cov : q < cov;
    bool bad = false;
    if (in) {
      const FarNode<NM>& f = node_at(0, q);
      bad = dist(f, g_near) < kFarTheta * f.s;
    }
    const uint64_t m = __ballot(bad);
    if (m == 0ull) break;
    const int far_bad = 64 - __builtin_clzll(m);   // leaves taken into the near range
    near_b = left ? near_b - far_bad : near_b + far_bad;
  }
  // a near range that reaches past the covered lines: no groups for the whole tile
  const int64_t stop = left ? min(near_b, cov) : max(near_b, cov);   // end of the groups
  const int64_t edge_b = left ? min(stop * kLeafLines, A.rec_n) : min(stop * kLeafLines, A.rec_n);
  const int64_t near_line = left ? max(end, min(near_b * kLeafLines, A.rec_n))
                                 : min(end, near_b * kLeafLines);
  if (!edge && lane == 0) {
    NearRange* nr = A.near + (int64_t)k * A.n_tiles + tile;
    if (left) nr->n0 = near_line;
    else nr->n1 = near_line;
  }

  __shared__ double red[kWavesPerWG][kWave];
  for (int p = 0; p < A.P; ++p) {
    const int64_t j = j0 + (int64_t)kWave * p + lane;
    const double v = A.grid[min(j, jl)];
    double sum = 0.0;
    auto add_node = [&](const FarNode<NM>& f) {
      const double rX = rcp64(v - 0.5 * (f.lo + f.hi));
      sum += moment_sum<NM>(f.A, f.s * rX, rX);
    };
    auto add_lines = [&](int64_t i0, int64_t i1) {
      for (int64_t i = i0; i < i1; ++i) sum += one_line<NM>(v, nu[i], recs[i]);
    };
    // the largest node at leaf position pos (outwards: its inner end) that stays within
    // `last` and is far from w; -1: not even the leaf is far
    auto pick = [&](int64_t pos, int64_t last, double w) {
      int l = -1;
      while (l + 1 < levels) {
        const int sh = 3 * (l + 1);
        const int64_t size = (int64_t)1 << sh;
        if ((pos & (size - 1)) != 0 || (left ? pos - size < last : pos + size > last)) break;
        const FarNode<NM>& f = node_at(l + 1, left ? (pos >> sh) - 1 : pos >> sh);
        if (dist(f, w) < kFarTheta * f.s) break;
        ++l;
      }
      return l;
    };
    if (!edge) {
      int64_t pos = near_b;
      while (left ? pos > cov : pos < cov) {
        const int l = pick(pos, cov, g_near);
        if (l < 0) {
          const int64_t q = left ? pos - 1 : pos;
          add_lines(q * kLeafLines, min((q + 1) * kLeafLines, A.rec_n));
          pos = left ? pos - 1 : pos + 1;
          continue;
        }
        const int sh = 3 * l;
        add_node(node_at(l, left ? (pos >> sh) - 1 : pos >> sh));
        pos = left ? pos - ((int64_t)1 << sh) : pos + ((int64_t)1 << sh);
      }
    } else {
      // lines [e, edge_b) (left) or [edge_b, e) (right) are inside this point's cut
      int64_t lo = left ? end : edge_b, hi = left ? edge_b : end;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const bool t = left ? v - nu[mid] <= cut : nu[mid] - v > cut;
        if (t) hi = mid;
        else lo = mid + 1;
      }
      const int64_t e = lo;
      if (left ? e < edge_b : e > edge_b) {
        const int64_t last = left ? (e + kLeafLines - 1) / kLeafLines : e / kLeafLines;
        // the leaf that this point's cut splits
        if (left) add_lines(e, min(last * kLeafLines, edge_b));
        else add_lines(max(last * kLeafLines, edge_b), e);
        int64_t pos = stop;
        while (left ? pos > last : pos < last) {
          const int l = pick(pos, last, v);
          if (l < 0) {
            const int64_t q = left ? pos - 1 : pos;
            add_lines(q * kLeafLines, min((q + 1) * kLeafLines, A.rec_n));
            pos = left ? pos - 1 : pos + 1;
            continue;
          }
          const int sh = 3 * l;
          add_node(node_at(l, left ? (pos >> sh) - 1 : pos >> sh));
          pos = left ? pos - ((int64_t)1 << sh) : pos + ((int64_t)1 << sh);
        }
      }
    }
    red[wv][lane] = sum;
    __syncthreads();
    if (wv == 0 && j <= jl) {
      double t = red[0][lane];
#pragma unroll
      for (int w = 1; w < kWavesPerWG; ++w) t += red[w][lane];
      A.out[(int64_t)k * A.n_grid + j] = t;
    }
    __syncthreads();
  }
}

hipError_t launch_far(const FarArgs& A, int moments, hipStream_t st) {
  if (A.n_items <= 0) return hipSuccess;
  const dim3 grid((unsigned)phys_workgroups(A.n_items)), block(kBlock);
  if (moments == kMomFp32)
    hipLaunchKernelGGL(xs_far_kernel<kMomFp32>, grid, block, 0, st, A);
  else
    hipLaunchKernelGGL(xs_far_kernel<kMomFp64>, grid, block, 0, st, A);
  return hipGetLastError();
}

}  // namespace xs
