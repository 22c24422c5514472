// Argument blocks shared by the kernels and the host runtime.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "physics.h"

namespace xs {

constexpr int kWave = 64;
constexpr int kWavesPerWG = 4;
constexpr int kBlock = kWave * kWavesPerWG;
constexpr int kMaxSplit = 256;
constexpr int kSelGroup = 4;   // tiles per main-contributor selection group
// Tiles of a workgroup that share one far-field expansion (one tile per wavefront).
constexpr int kGroup = kWavesPerWG;
// Device scratch of the allocation-free entry point (one array per device, kernels.hip).
constexpr size_t kNoAllocScratchBytes = (size_t)256 << 20;
constexpr int kPtsPerFill = 64;   // P-T pairs per fill launch (passed as kernel arguments)

struct LinesDev {
  const double* nu0;
  const float* A;
  const float* E;
  const float* gam;
  const float* nT;
  const uint16_t* g;
  const uint16_t* J;   // lower-state J (nullptr: 0 for every line)
  int64_t n;
};

// Per (line, P-T point) parameters written by the parameter kernel: the cutoff half-width,
// 1/b_D, the profile scale S/(b_D sqrt(pi)) and y = gamma_L/b_D (all FP64, 32 bytes).
struct LineRec {
  double cut, ib, sc, y;
};

// Tree of line groups over the record range [rec_lo, rec_lo + rec_n) (far_tree.h): level l
// has cnt[l] nodes from index off[l], n_nodes in all, one array of them per (P, T) point.
constexpr int kPointGroup = 8;   // grid points per wavefront of the point kernel
constexpr int kTreeLevels = 7;
// A group of points is cut in runs at a gap that holds more lines than this beyond the near
// ranges beside it, as they cost more than the runs' own searches: one gap of many small steps
// (more than half of the group), or steps that are all that wide (1050 lines/cm^-1, steps of 1 cm^-1:
// 509 us as one group, 729 in runs; steps of 10 cm^-1: 657 and 646).
constexpr int kGapLines = 1024, kStepLines = 8192;
struct TreeDims {
  int64_t off[kTreeLevels];
  int64_t cnt[kTreeLevels];
  int64_t n_nodes;
  int levels;             // levels in use
};
// Lines [n0, n1) of the record range that a tile's own kernel walks; the far kernel takes
// the others.
struct NearRange {
  int64_t n0, n1;
};

// The lines of every whole block of kCutBlock lines (a tree node of level kCutLevel) in order
// of falling cut, 16 to a group (far_tree.h): per (P, T) point and block the sorted keys
// (cut, line of the block) and per group the moments of the lines up to its end.
constexpr int kCutLevel = 3;
constexpr int kCutBlock = 1024;
struct CutOrder {
  int blocks;             // per (P, T) point; 0: cuts are one, or too few lines
  uint32_t* keys;         // [n_pt][blocks][kCutBlock]
  double* pre;            // [n_pt][blocks][kCutBlock / 16][moments]
};

struct ParamArgs {
  LinesDev L;
  SpeciesDev sp;
  CutDev cut;
  const double* pts;      // [n_pts][2] = (P bar, T K), whole table
  int pt0, n_pt;          // this batch: points pt0 .. pt0 + n_pt - 1
  int64_t lo, n;          // line range [lo, lo + n)
  LineRec* out;           // [n_pt][n]
  double* nodes;          // tree nodes [n_pt][dims.n_nodes] (nullptr: no tree)
  TreeDims dims;
  int moments;            // kMomFp32 or kMomFp64
  PtBounds* bounds;       // [n_pt] (with a tree)
  CutOrder order;         // blocks == 0: none
};

// The far kernel: per (tile, P-T point) the sum over the lines outside the tile's near
// range, and that range.
struct FarArgs {
  LinesDev L;
  SpeciesDev sp;
  double cut;             // the fixed cut
  const double* grid;
  int64_t n_grid;
  const double* pts;      // [n_pts][2], whole table
  int pt0, n_pt;          // this batch
  int P;                  // points per lane of the tile kernel (a tile is 64 P points)
  int64_t n_items;        // tiles issued * n_pt
  const int* tile_order;  // issue order of the tiles (nullptr: ascending)
  int64_t n_tiles;        // tiles of the whole grid
  const LineRec* recs;
  int64_t rec_lo, rec_n;
  const double* nodes;
  TreeDims dims;
  double* out;            // [n_pt][n_grid]
  NearRange* near;        // [n_pt][n_tiles]
};

// The point kernel: whole sums at kPointGroup neighbouring grid points per wavefront.
struct PointArgs {
  LinesDev L;
  CutDev cut;
  const PtBounds* bounds; // [n_pt]
  const double* grid;
  int64_t n_grid;
  int pt0, n_pt;          // points of this launch
  int split;              // parts of a group's work, each a wavefront of its own
  int64_t g0, n_groups;   // groups of kPointGroup grid points
  const LineRec* recs;    // [n_pt][rec_n]
  int64_t rec_lo;
  int rec_n;
  const double* nodes;
  TreeDims dims;
  CutOrder order;         // of this launch's first point
  void* out;              // split == 1: sigma rows [n_pts][n_grid] (row pt0 + k); else
                          // partials [n_pt][split][n_grid] (double)
  int out_f32;
  int runs;               // the grid has gaps of many lines (kGapLines)
  float l1_eps;           // error budget of the shifted Lorentzian
};

struct TileArgs {
  LinesDev L;
  SpeciesDev sp;
  CutDev cut;
  const double* grid;
  int64_t n_grid;
  const double* pts;      // [n_pts][2], whole table
  int pt0, n_pt;          // this batch
  int split;
  int group;              // 1: a work item is one tile (one wavefront); kGroup: a work
                          // item is kGroup neighbouring tiles (one workgroup)
  int64_t n_tiles;        // units issued: tiles, or groups of kGroup tiles
  int64_t n_items;        // n_tiles * n_pt * split
  int64_t n_wg;           // logical workgroups (ceil(n_items / 4), or n_items grouped)
  const int* tile_order;  // issue order of the units (nullptr: ascending)
  const LineRec* recs;    // [n_pt][rec_n] records of lines [rec_lo, rec_lo + rec_n)
  int64_t rec_lo, rec_n;
  double* out;            // split == 1: sigma rows [n_pts][n_grid] (row pt0 + k);
                          // else partials [n_pt][split][n_grid] of this batch
  int out_f32;            // split == 1 only: out holds float rows instead of double
  unsigned long long* counts;  // count kernel only: [n_pts][kNEvalTiers]
  // main-contributor selection (nullptr: off): per (P, T) point of the batch and group of
  // kSelGroup neighbouring tiles (tile / kSelGroup), the contribution bound below which a
  // line is dropped, [n_pt][tau_stride]
  double* tau;
  int64_t tau_stride;     // groups of the whole grid
  double select_eps;      // select kernel: the allowed relative error
  // far field by moments (nullptr: every line of the window is walked here): the lines each
  // tile walks, [n_pt][near_stride], and the others' sums, [n_pt][n_grid], added here when
  // split == 1 (else by the reduction)
  const NearRange* near;
  int64_t near_stride;
  const double* far;
  int chunks;             // FP64 path without near: chunks of lines by their moments
  // error budget of the shifted forms (shifted_lorentz_ok, dshift_ok) and the far-line
  // threshold kappa (far_line_ok) for that budget
  float l1_eps, far_kappa;
};

// Launchers (kernels.hip). phys_wg = number of workgroups launched: n_wg rounded up to a
// multiple of 8 * 16 (whole XCD blocks).
inline int64_t phys_workgroups(int64_t n_wg) { return (n_wg + 127) / 128 * 128; }
// The launch grid of n workgroups of at most 1024 threads: a dimension holds at most 2^32 - 1
// threads, so more than kMaxGridX of them go into rows of kMaxGridX (a multiple of 128; the last
// row may hold workgroups past n, which have no work).
constexpr int64_t kMaxGridX = (int64_t)1 << 21;
inline dim3 wg_grid(int64_t n) {
  return n <= kMaxGridX ? dim3((unsigned)n)
                        : dim3((unsigned)kMaxGridX, (unsigned)((n + kMaxGridX - 1) / kMaxGridX));
}
hipError_t launch_params(const ParamArgs& A, hipStream_t st);
hipError_t launch_tile(const TileArgs& A, int P, bool f64, int W, hipStream_t st,
                       int64_t phys_wg);
hipError_t launch_count(const TileArgs& A, int P, hipStream_t st, int64_t phys_wg);
// one wavefront per (group of 4 tiles, P-T point), A.n_tiles groups: writes A.tau
hipError_t launch_select(const TileArgs& A, int P, bool wide, hipStream_t st);
// per points-per-lane instantiations of the tile kernel (tile_p*.hip)
hipError_t launch_tile_p1(const TileArgs& A, bool f64, int W, hipStream_t st, dim3 grid);
hipError_t launch_tile_p2(const TileArgs& A, bool f64, int W, hipStream_t st, dim3 grid);
hipError_t launch_tile_p4(const TileArgs& A, bool f64, int W, hipStream_t st, dim3 grid);
hipError_t launch_tile_p8(const TileArgs& A, bool f64, int W, hipStream_t st, dim3 grid);
// the moments of every level above the leaves (launch_params writes those)
hipError_t launch_tree_up(const ParamArgs& A, hipStream_t st);
// the blocks' orders by cut (A.order)
hipError_t launch_cut_order(const ParamArgs& A, hipStream_t st);
hipError_t launch_far(const FarArgs& A, int moments, hipStream_t st);
hipError_t launch_point(const PointArgs& A, int moments, hipStream_t st);
// out: float rows when out_f32, else double rows; far (may be nullptr): one more partial
hipError_t launch_reduce(const double* part, const double* far, void* out, int out_f32,
                         int64_t n_grid, int n_pts, int split, hipStream_t st);
// collision-induced absorption: block k (nodes [off[k], off[k+1]) of nu, alpha) linearly
// interpolated onto the grid, zero outside the block, out[k][j]
hipError_t launch_cia(const double* grid, int64_t n_grid, const int64_t* off, int n_blocks,
                      const double* nu, const double* alpha, double* out, hipStream_t st);
hipError_t launch_eval_voigt(const double* x, const double* y, int64_t n, int f64,
                             double* out, hipStream_t st);
hipError_t launch_fill_u64(unsigned long long* p, int64_t n, hipStream_t st);
// dst[0 .. 2 n) = pairs[0 .. 2 n), the values passed as kernel arguments (no copy from
// host memory), kPtsPerFill pairs per launch
hipError_t launch_fill_pts(double* dst, const double* pairs, int64_t n, hipStream_t st);
// Device address of the allocation-free scratch array on the current device (called once
// per device, with that device current).
hipError_t noalloc_scratch_address(void** out);
// g[j] = a + j * h (FP64, one rounding per operation, no contraction)
hipError_t launch_fill_uniform(double* g, int64_t n, double a, double h, hipStream_t st);

}  // namespace xs
