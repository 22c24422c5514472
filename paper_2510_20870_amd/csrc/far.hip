// Far field by moments of line groups (far_tree.h): the levels of the tree above its leaves,
// and the far kernel, which sums for every grid tile the lines outside its near range. The
// tile kernel walks the near range; this pair serves the (P, T) points whose lines are so
// broad that a near range spans many tiles (there the tile polynomial takes most of it). The
// others go by the point kernel (point.hip).
//
// Section "Functionality of pyROX" (bullets "Compute line profiles", "Combine and save"): the
// sum over every line inside the cutoff; here the lines far from a grid point enter group by
// group, with the same cutoff test per (line, point) pair.
#include "far_tree.h"
#include "tile_kernel.h"

namespace xs {

// n!, n <= kMomFp64
struct Factorials {
  double v[kMomFp64 + 1];
};
constexpr Factorials make_factorials() {
  Factorials f{};
  f.v[0] = 1.0;
  for (int n = 1; n <= kMomFp64; ++n) f.v[n] = f.v[n - 1] * n;
  return f;
}
constexpr Factorials kFactorial = make_factorials();

// One parent from its n children (nodes q0 .. q0 + n - 1 of the level below). A child's
// moments move to the parent's centre and scale by the binomial theorem, which for moments
// divided by m! is a plain product of series: T'_m / m! = sum_k (R^k A_k / k!) (D^(m-k) /
// (m-k)!), D the distance of the centres and R the child's scale, in parent scales. One thread
// holds the whole parent in registers, so the term products (136 for 16 moments) are a
// straight run with no table, no shared memory and neighbouring threads reading
// neighbouring nodes.
template <int NM>
__device__ __forceinline__ void merge_node(const double* nodes, int64_t q0, int n, double kb,
                                           double* to) {
  const NodeRef<NM, const double> first{nodes + node_pos<NM>(q0)};
  const double lo = first.lo();
  const double hi = NodeRef<NM, const double>{nodes + node_pos<NM>(q0 + n - 1)}.hi();
  double g = first.at(kNodeG);
  for (int i = 1; i < n; ++i)
    g = fmax(g, NodeRef<NM, const double>{nodes + node_pos<NM>(q0 + i)}.at(kNodeG));
  const double h = 0.5 * (hi - lo), c = 0.5 * (lo + hi);
  const double s = sqrt(fma(h, h, g * g)) + far_beta<NM>() * (kb * hi);
  const double is = 1.0 / s;
  double sum[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) sum[m] = 0.0;
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    const NodeRef<NM, const double> f{nodes + node_pos<NM>(q0 + i)};
    const double D = (f.c() - c) * is, R = f.s() * is;
    double a[NM], e[NM];   // R^k A_k / k! (k = index + 1), D^j / j!
    double pr = R, pd = 1.0;
#pragma unroll
    for (int k = 0; k < NM; ++k) {
      a[k] = pr * f.at(kNodeA + k);
      e[k] = pd;
      pr *= R * (1.0 / (k + 2));
      pd *= D * (1.0 / (k + 1));
    }
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int k = 0; k <= m; ++k) sum[m] = fma(a[k], e[m - k], sum[m]);
  }
  const NodeRef<NM, double> p{to};
  p.at(kNodeLo) = lo;
  p.at(kNodeHi) = hi;
  p.at(kNodeS) = s;
  p.at(kNodeG) = g;
#pragma unroll
  for (int m = 0; m < NM; ++m) p.at(kNodeA + m) = sum[m] * kFactorial.v[m + 1];
}

// Three levels at once: a workgroup takes 4 kBlock nodes of level l, writes their parents, one
// per thread, and, where those levels exist, the two levels above those. The first of the
// three levels reads nearly all the bytes; the other two run on a quarter and a sixteenth of
// the threads, whose latency (about 900 dependent-free instructions each) is what a small
// list waits for.
template <int NM>
__global__ __launch_bounds__(kBlock) void xs_tree_up_kernel(ParamArgs A, int l) {
  const int k = blockIdx.y;
  double* nodes = A.nodes + (int64_t)k * A.dims.n_nodes * node_fields<NM>();
  const double kb = A.bounds[k].kb;
  int per = kBlock;   // parents of a whole workgroup
#pragma unroll 1
  for (int up = l + 1; up <= l + 3 && up < A.dims.levels; ++up, per /= kArity) {
    const int64_t q = (int64_t)blockIdx.x * per + threadIdx.x;
    if ((int)threadIdx.x < per && q < A.dims.cnt[up]) {
      const int n = (int)min((int64_t)kArity, A.dims.cnt[up - 1] - q * kArity);
      merge_node<NM>(nodes, A.dims.off[up - 1] + q * kArity, n, kb,
                     nodes + node_pos<NM>(A.dims.off[up] + q));
    }
    __syncthreads();   // (the next level reads what this one wrote)
  }
}

hipError_t launch_tree_up(const ParamArgs& A, hipStream_t st) {
  if (A.n <= 0 || A.n_pt <= 0) return hipSuccess;
  for (int l = 0; l + 1 < A.dims.levels; l += 3) {
    const dim3 grid((unsigned)((A.dims.cnt[l + 1] + kBlock - 1) / kBlock), (unsigned)A.n_pt);
    const dim3 block(kBlock);
    if (A.moments == kMomFp32)
      hipLaunchKernelGGL(xs_tree_up_kernel<kMomFp32>, grid, block, 0, st, A, l);
    else
      hipLaunchKernelGGL(xs_tree_up_kernel<kMomFp64>, grid, block, 0, st, A, l);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Values of the lane whose index differs by the mask kX: inside a row of 16 by DPP (4 as 7
// then 3).
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}
template <int kX>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (kX == 1) return dpp_u32<kRowX1>(v);
  else if constexpr (kX == 2) return dpp_u32<kRowX2>(v);
  else if constexpr (kX == 4) return dpp_u32<0x1b>(dpp_u32<kRowX7>(v));
  else if constexpr (kX == 8) return dpp_u32<kRowX8>(v);
  else return (uint32_t)__shfl_xor((int)v, kX);
}
// v of the lane d below inside the row of 16, 0 where there is none (row_shr:d)
template <int d>
__device__ __forceinline__ double row_below(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = dpp_u32<0x110 + d>((uint32_t)u), hi = dpp_u32<0x110 + d>((uint32_t)(u >> 32));
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

// One stage of the bitonic network over e = 16 lane + r: e against e ^ j, in runs of w.
template <int w, int j>
__device__ __forceinline__ void sort_stage(uint32_t (&v)[16], int lane) {
  if constexpr (j >= 16) {
    const bool big = ((lane & (j / 16)) == 0) == ((lane & (w / 16)) == 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t o = lane_xor<j / 16>(v[r]);
      v[r] = big ? max(v[r], o) : min(v[r], o);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if ((r & j) != 0) continue;
      const bool falling = w < 16 ? (r & w) == 0 : (lane & (w / 16)) == 0;
      const uint32_t hi = max(v[r], v[r + j]), lo = min(v[r], v[r + j]);
      v[r] = falling ? hi : lo;
      v[r + j] = falling ? lo : hi;
    }
  }
  if constexpr (j > 1) sort_stage<w, j / 2>(v, lane);
}

// The order by cut of one block (far_tree.h), by one wavefront: lane i holds sorted places
// 16 i to 16 i + 15 in registers (a bitonic network; strides below 16 stay in the lane), then
// the moments of its 16 lines about the block's centre, and a scan over the lanes adds those
// before it. What bounds it is reading the records twice, in order for the cuts and gathered
// for the moments: 2.1e6 lines x 12 (P, T) points take 676 us (0.8 GB of records, 0.4 GB
// written; exchanges by DPP instead of LDS gave 30 us of that). With it the point kernel takes
// 3.1 ms instead of 6.2 on 25147 grid points: up to 1.7e5 lines lie between a point's
// smallest and largest cut, and were tested and summed one by one.
template <int NM>
__global__ __launch_bounds__(kBlock) void xs_cut_order_kernel(ParamArgs A) {
  constexpr int kPer = kCutBlock / kWave;
  static_assert(kPer == kLeafLines && kCutBlock == kLeafLines << (kArityBits * kCutLevel),
                "a lane is a group, a block is a node");
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int blk = blockIdx.x * kWavesPerWG + wv, k = blockIdx.y;
  if (blk >= A.order.blocks) return;
  // (the point kernel asks for no order where every line's cut is the cap)
  if (A.cut.mult * voigt_fwhm(A.bounds[k].gmin, 0.0) >= A.cut.cut * (1.0 + 1e-9)) return;
  const int64_t l0 = (int64_t)blk * kCutBlock;
  const LineRec* recs = A.out + (int64_t)k * A.n + l0;
  const double* nu = A.L.nu0 + A.lo + l0;
  uint32_t v[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) v[r] = cut_key(recs[r * kWave + lane].cut, A.cut.cut, r * kWave + lane);
  sort_stage<2, 1>(v, lane);
  sort_stage<4, 2>(v, lane);
  sort_stage<8, 4>(v, lane);
  sort_stage<16, 8>(v, lane);
  sort_stage<32, 16>(v, lane);
  sort_stage<64, 32>(v, lane);
  sort_stage<128, 64>(v, lane);
  sort_stage<256, 128>(v, lane);
  sort_stage<512, 256>(v, lane);
  sort_stage<1024, 512>(v, lane);
  const int64_t at = (int64_t)k * A.order.blocks + blk;
  uint4* keys = (uint4*)(A.order.keys + at * kCutBlock + lane * kPer);
#pragma unroll
  for (int r = 0; r < kPer; r += 4) keys[r / 4] = make_uint4(v[r], v[r + 1], v[r + 2], v[r + 3]);
  const NodeRef<NM, const double> f =
      node_at<NM>(A.nodes + (int64_t)k * A.dims.n_nodes * node_fields<NM>(), A.dims, kCutLevel, blk);
  const double c = f.c(), is = 1.0 / f.s();
  double sum[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) sum[m] = 0.0;
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const int i = (int)(v[r] & (kCutBlock - 1));
    const LineRec lr = recs[i];
    const double b = rcp64(lr.ib), bs = b * is;
    double M[NM];
    // (S/pi from the record's S / (b sqrt(pi)))
    line_moments<NM>(lr.sc * b * kInvSqrtPi, (nu[i] - c) * is, lr.y * bs, 0.5 * bs * bs, M);
#pragma unroll
    for (int m = 0; m < NM; ++m) sum[m] += M[m];
  }
  double2* pre = (double2*)(A.order.pre + (at * kWave + lane) * NM);
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    double t = sum[m];
    t += row_below<1>(t);
    t += row_below<2>(t);
    t += row_below<4>(t);
    t += row_below<8>(t);
    // the rows before this one
    const double r0 = lane_value(t, 15), r1 = lane_value(t, 31), r2 = lane_value(t, 47);
    t += lane < 16 ? 0.0 : lane < 32 ? r0 : lane < 48 ? r0 + r1 : r0 + r1 + r2;
    sum[m] = t;
  }
#pragma unroll
  for (int m = 0; m < NM; m += 2) pre[m / 2] = make_double2(sum[m], sum[m + 1]);
}

hipError_t launch_cut_order(const ParamArgs& A, hipStream_t st) {
  if (A.order.blocks <= 0 || A.n_pt <= 0) return hipSuccess;
  const dim3 grid((unsigned)((A.order.blocks + kWavesPerWG - 1) / kWavesPerWG), (unsigned)A.n_pt);
  const dim3 block(kBlock);
  if (A.moments == kMomFp32)
    hipLaunchKernelGGL(xs_cut_order_kernel<kMomFp32>, grid, block, 0, st, A);
  else
    hipLaunchKernelGGL(xs_cut_order_kernel<kMomFp64>, grid, block, 0, st, A);
  return hipGetLastError();
}

// Far kernel. One workgroup per (tile, P-T point): wavefronts 0 and 1 take the groups left
// and right of the near range that are inside the cut of every point of the tile (the same
// nodes for all lanes), wavefronts 2 and 3 the lines beyond, up to each point's own cut
// (a walk over nodes per lane). What bounds it is the latency of a node's loads and of its
// Horner chain: the node counts grow with the logarithm of the window, not with its lines.
//
// Near range: from the tile outwards by theta times the list's largest widths there, then
// over the leaves up to the last of the leaves nearby that are not far from the whole tile
// (|nu - c| < theta s for some point); each 64-leaf group is tested at once, and the range
// ends at the first group of far leaves. (Taking the widths from the leaves alone costs a
// dependent step per 64 leaves: 1.6 ms instead of 0.1 at 100 bar on the 1e9-line list.)
template <int NM>
__global__ __launch_bounds__(kBlock) void xs_far_kernel(FarArgs A) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = logical_wg();
  if (item >= A.n_items) return;   // the whole workgroup
  const int k = (int)(item % A.n_pt);
  const int64_t tile = A.tile_order ? (int64_t)A.tile_order[item / A.n_pt] : item / A.n_pt;
  const int64_t j0 = tile * kWave * A.P;
  const int64_t jl = min(j0 + (int64_t)kWave * A.P, A.n_grid) - 1;
  const double g0 = A.grid[j0], g1 = A.grid[jl];
  const int pt = A.pt0 + k;
  const PtConst pc = make_pt(A.sp, A.pts[2 * pt], A.pts[2 * pt + 1]);
  const double kb = pc.dopp / kCLight;
  // the list's largest Lorentz width here
  const double gmax = A.sp.gam_max * pc.pfac * fmax(pow(pc.tratio, A.sp.n_min),
                                                    pow(pc.tratio, A.sp.n_max));
  const double cut = A.cut;
  const double* nu = A.L.nu0 + A.rec_lo;
  const LineRec* recs = A.recs + (int64_t)k * A.rec_n;
  const double* nodes = A.nodes + (int64_t)k * A.dims.n_nodes * node_fields<NM>();
  using Node = NodeRef<NM, const double>;
  const int levels = A.dims.levels;
  const bool left = (wv & 1) == 0, edge = wv >= 2;
  auto node = [&](int l, int64_t q) -> Node { return node_at<NM>(nodes, A.dims, l, q); };
  // signed distance from v outwards to the node's centre
  auto dist = [&](const Node& f, double v) { return left ? v - f.c() : f.c() - v; };
  const double g_near = left ? g0 : g1;   // the tile's point nearest to this side's lines

  // this side's ranges, in lines of the record range: near boundary (a leaf boundary),
  // lines inside the cut of every point up to `cov` (leaf boundary), reachable up to `end`
  int64_t near_b, cov, end;   // near_b, cov: leaf indices
  const double reach = kFarTheta * (gmax + far_beta<NM>() * kb * g_near);
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
      const Node f = node(0, q);
      bad = dist(f, g_near) < kFarTheta * f.s();
    }
    const uint64_t m = __ballot(bad);
    if (m == 0ull) break;
    const int far_bad = 64 - __builtin_clzll(m);   // leaves taken into the near range
    near_b = left ? near_b - far_bad : near_b + far_bad;
  }
  // a near range that reaches past the covered lines: no groups for the whole tile
  const int64_t stop = left ? min(near_b, cov) : max(near_b, cov);   // end of the groups
  const int64_t edge_b = min(stop * kLeafLines, A.rec_n);
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
    auto add_node = [&](const Node& f) {
      const double rX = rcp64(v - f.c()), t = f.s() * rX;
      double a = f.at(kNodeA + NM - 1);
#pragma unroll
      for (int m = NM - 2; m >= 0; --m) a = fma(a, t, f.at(kNodeA + m));
      sum = fma(a * t, rX, sum);
    };
    auto add_lines = [&](int64_t i0, int64_t i1) {
      for (int64_t i = i0; i < i1; ++i) sum += one_line<NM>(v, nu[i], recs[i]);
    };
    // the largest node at leaf position pos (outwards: its inner end) that stays within
    // `last` and is far from w; -1: not even the leaf is far
    auto pick = [&](int64_t pos, int64_t last, double w) {
      int l = -1;
      while (l + 1 < levels) {
        const int sh = kArityBits * (l + 1);
        const int64_t size = (int64_t)1 << sh;
        if ((pos & (size - 1)) != 0 || (left ? pos - size < last : pos + size > last)) break;
        const Node f = node(l + 1, left ? (pos >> sh) - 1 : pos >> sh);
        if (dist(f, w) < kFarTheta * f.s()) break;
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
        const int sh = kArityBits * l;
        add_node(node(l, left ? (pos >> sh) - 1 : pos >> sh));
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
          const int sh = kArityBits * l;
          add_node(node(l, left ? (pos >> sh) - 1 : pos >> sh));
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
  const dim3 grid = wg_grid(phys_workgroups(A.n_items)), block(kBlock);
  if (moments == kMomFp32)
    hipLaunchKernelGGL(xs_far_kernel<kMomFp32>, grid, block, 0, st, A);
  else
    hipLaunchKernelGGL(xs_far_kernel<kMomFp64>, grid, block, 0, st, A);
  return hipGetLastError();
}

}  // namespace xs
