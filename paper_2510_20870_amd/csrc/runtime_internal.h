// Internal state of a context (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <set>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/xsec.h"
#include "far_tree.h"
#include "kernel_args.h"

namespace xs {

struct Scratch {
  void* ptr = nullptr;
  size_t cap = 0;
};

struct LinesRes {
  LinesDev dev{};
  SpeciesDev sp{};
  void* base = nullptr;     // one device allocation holding every array
  size_t bytes = 0;
  size_t n = 0;
  std::atomic<int> refs{0}; // pending serving requests and live graphs
  std::vector<double> q_T_host, q_val_host;
  std::vector<double> sample;   // nu0 of every kSampleStride-th line (host index)
  double nu_last = 0.0;         // nu0 of the last line
};

constexpr int64_t kSampleStride = 1024;
// Longest line range of one work item of a served request (its default split keeps items
// at or under it, so that a new request's kernels find free wavefront slots quickly).
constexpr int64_t kServeItemLines = 4096;

// Far field by moments: from kMomentLines lines with a fixed cut (those within the cut where the
// list is densest, and those that a tile of 64 points spans besides: tile_lines); with fewer, for
// a fixed cut and no wide point (kWideSteps), from kMomentList lines in the list. There a call
// that does not fill the device wins by its shorter chains, a larger one only where a window
// holds so many lines that walking them costs more than the point kernel's searches and sums
// (some 0.5 ns per point): beyond kMomentGroups1 groups of points in all from kMomentLines1 lines on, beyond kMomentGroups2 from kMomentLines2.
// Measured with a fixed cut (us, tile kernel alone / by moments; one (P, T) point of 3e4, 2e5, 1e6
// grid points): 100 lines in the window 68 / 41, 151 / 140, 251 / 550; 500 lines 82 / 46,
// 181 / 173, 377 / 687; 2000 lines 147 / 51, 255 / 201, 748 / 810; 5000 lines 217 / 64, 401 / 225,
// 1502 / 943; 15000 lines 404 / 79, 848 / 275, 3787 / 1466; tables of 8 x 1e5, 24 x 1e5 and
// 8 x 4e5: 3000 lines 612 / 498, 1075 / 1332, 1066 / 1726; 5000 lines 936 / 535, 1696 / 1438,
// 1553 / 1857; 8000 lines 1412 / 582, 2640 / 1599, 2284 / 2017. A wide point has nearly all lines
// beside it. On the FP64 path only from kMomentLines64 lines on (28 moments per leaf: 40 points, 100
// lines 27 / 35, 300 lines 31 / 35, 600 lines 39 / 37), which then holds for every size
// (4 x 3.3e5 points, 730 lines 547 / 445). The lines beside a tile weigh 16-fold in the two limits
// (3.1e5 points of steps of 0.006 cm^-1, 1890 lines within 3 cm^-1: 657 / 339).
constexpr int64_t kMomentLines = 16384, kMomentList = 512, kMomentLines64 = 384;
constexpr int64_t kMomentLines1 = 3072, kMomentGroups1 = 25000;
constexpr int64_t kMomentLines2 = 6144, kMomentGroups2 = 125000;
// With a FWHM cut only from kMomentLines lines within the cap (6550 lines go from 224 to 417: those
// that only some points reach are far too few per block). The orders by cut make the chain of
// launches longer, and what tiles cost follows from the lines within their own cuts: so by moments
// from kFwhmOwn1 lines within the widest of these on (and in a tile's span) up to kFwhmGroups1
// groups of points in all (FP64: kFwhmOwn64 up to kFwhmGroups64, then kFwhmOwn3), from
// kFwhmOwn2 on more, where every line's cut is the cap at some point (53000 lines at 100 bar, 64
// points 230 / 105), and where the cap holds so many that the parameters of all of them are what
// counts. With a given split from kFwhmLines1 within the cap, whatever the points. Measured (us,
// tiles / moments; one (P, T) point at 1000 K of 0.001, 0.3, 1, 3 bar, for which the widest of the lines' own cuts hold 0.012,
// 0.15, 0.5 and 1 times the lines within the cap): FP32, 17000 lines, 1349 points 45 / 107, 59 / 113,
// 102 / 127, 158 / 116; 40000 points 101 / 91, 124 / 134, 140 / 210, 187 / 257; 400000 points
// 242 / 288, 307 / 644, 509 / 1117, 825 / 1096; 50000 lines, 1349 points 58 / 115, 112 / 126,
// 227 / 122, 396 / 138; 40000 points 120 / 103, 213 / 222, 244 / 286, 390 / 360; 400000 points
// 359 / 332, 570 / 1167, 1162 / 1214, 2112 / 1485; 200000 lines, 400000 points 848 / 423,
// 1704 / 1349, 4126 / 2078, 8036 / 3194. FP64, 17000 lines, 1349 points 49 / 115, 85 / 140, 91 / 190,
// 146 / 160; 400000 points 300 / 502, 970 / 1071, 1729 / 1828, 2538 / 1651; 50000 lines, 400000 points
// 612 / 566, 1722 / 1972, 3277 / 1789, 5317 / 2235. At 9000 cm^-1, where the Doppler widths make the
// cuts, 4300 of 30000 lines, 629 and 9508 points FP32 173 / 79, 210 / 86, FP64 111 / 124, 251 / 145.
constexpr int64_t kFwhmGroups64 = 512, kFwhmGroups1 = 2048, kFwhmGroups2 = 16384;
constexpr int64_t kFwhmLines1 = 32768, kFwhmLines2 = 65536;
constexpr int64_t kFwhmOwn1 = 4096, kFwhmOwn2 = 20480, kFwhmOwn64 = 16384, kFwhmOwn3 = 3072;
// Small calls of that kind keep the tree low, as each three of its levels are a launch of some
// 20 us: the fewest levels that leave at most kTopNodes nodes in a window, for at most
// kFewGroups groups of points.
constexpr int64_t kFewGroups = 16384, kTopNodes = 512;
// (P, T) points whose near range reaches this many grid steps on each side go by tiles, whatever
// the tile's size (with 4 or 8 points per lane a limit of so many tiles kept points at 50 bar in
// the point kernel: 10000 points, 3750 lines/cm^-1, 1057 us, by tiles of 4 points per lane 588).
constexpr double kWideSteps = 384.0;
// Where the lines' cuts differ (FWHM), broad points go by tiles over whole windows: those with at
// least this part of the lines within their own widest cut in the near range (40600 lines/cm^-1,
// 12356 points, us by tiles / point kernel: 1 bar 2573 / 1107, 3 bar 1940 / 1020, 10 bar 744 / 4188,
// 30 bar 548 / 8250; the part is 0.07 at 3 bar, 0.22 at 10).
constexpr double kNearAll32 = 0.125;
// On the FP64 path only those whose near range holds at least this part, and so many lines (24
// points in turn, 2855 lines, 9052 grid points 1727 us, 405 by the point kernel): its tiles gain
// little from the far field's polynomial. (Tiles / point kernel, us: 17000 lines in the window,
// 800 points at 3, 30, 60, 100 bar 187 / 89, 178 / 112, 178 / 136, 158 / 151; 5000 points at 60 and
// 100 bar 224 / 210, 235 / 265; 50000 lines, 2000 points 256 / 305, 267 / 399; 1e5 points at 20 and
// 100 bar 1995 / 1776, 7177 / 7727. The near range is 0.6 of the cut at 60 bar.)
constexpr double kNearAll64 = 0.8, kNearLines64 = 16384.0;
// Main-contributor selection's thresholds by workgroups of 16 waves from so many lines in a window
// on (sampled, so rather more than there are) or up to so many groups of tiles, else of 4 waves.
// Whole calls, us, 4 / 16 waves: 5 lines, 235 groups, 8 (P, T) points 105 / 116, 586 groups 137 / 165;
// 500 lines 187 / 200, 284 / 320; 1800 lines, 195 groups 131 / 126, 4 groups 67 / 61; 5000 lines 223 / 203,
// 405 / 390. The rule looks at the grid and the list alone, as the thresholds' rounding follows the
// workgroup.
constexpr int64_t kSelLines = 3072, kSelGroups = 64;
// Tables of up to this many groups of points in all go one way where their points would go two
// ways in turn (over whole windows a quarter as many: 24 points of the table with FWHM cuts, 1180
// lines/cm^-1 on 715 points 443 us in runs, 1071 as one).
constexpr int64_t kTurnGroups = 4096;
// Grids with gaps of many lines keep broad points in the point kernel up to this many points.
constexpr size_t kSeamPoints = 65536;
// Of a grid of one point: those with this many lines in the near range. (1050 lines/cm^-1: 0.1 bar
// 70 us by the point kernel, 209 by tiles; 30 bar 83 and 92; 100 bar, 47000 near lines, 134 and 82)
constexpr double kWideLines = 32768.0;

struct GridRes {
  double* d = nullptr;
  size_t n = 0;
  size_t bytes = 0;
  double first = 0.0, last = 0.0;   // host copies of the end points
  double max_step = 0.0;            // the widest gap between neighbouring points,
  size_t max_at = 0;                // from this point to the next
  std::vector<double> host;         // host copy of the grid
  std::atomic<int> refs{0};         // pending serving requests and live graphs
};

// How a (P, T) point of a call by moments is summed: the point kernel, tiles over the near ranges
// beside the far kernel's sums, or tiles over whole windows (without the tree).
enum PointWay : uint8_t { kPoint = 0, kTileNear = 1, kTileWhole = 2 };

struct Plan {
  int P = 4;               // grid points per lane (tile = 64 P points)
  int split = 1;           // line splits per tile
  int W = 0;               // occupancy target of the tile kernel (0, 3 or 4 waves/SIMD)
  int64_t n_tiles = 0;
  int group = 1;           // tiles per work item (kGroup: grouped far field)
  int64_t n_units = 0;     // units of the issue order: tiles, or groups of `group` tiles
  int64_t rec_lo = 0;      // lines [rec_lo, rec_lo + rec_n) can reach the grid
  int64_t rec_n = 0;
  int npts = 0;
  int pt_batch = 1;        // (P, T) points per parameter/tile launch pair
  std::vector<int> tile_order;   // units by decreasing estimated work
  std::vector<int64_t> tile_cost;  // estimated lines of each unit (x 1024): in its window, or
                                   // by moments near it
  bool tuned = false;              // launch shape from the tuning cache
  double select_eps = 0.0;         // main-contributor selection (0: off)
  bool wide_select = false;        // thresholds by workgroups of 16 waves
  // Far field by moments (far_tree.h): the tree over the records, 0 moments: off.
  int moments = 0;
  std::vector<uint8_t> by_tile;   // per (P, T) point: a PointWay
  bool any_tile = false;
  bool runs = false;              // the grid has gaps of many lines (kGapLines)
  int tile_split = 1;             // line splits of the points by tiles
  // the point kernel's groups of points in a tile of 64 P points
  int64_t groups_per_tile() const {
    return std::max<int64_t>(1, std::min<int64_t>(kWave * P, n_grid + kPointGroup - 1) / kPointGroup);
  }
  std::vector<uint8_t> chunks;    // per (P, T) point: FP64 tile kernel, chunks of lines by their
  bool any_chunks = false;        // moments
  int max_split() const { return any_tile && tile_split > split ? tile_split : split; }
  TreeDims dims{};
  int cut_blocks = 0;             // blocks ordered by cut (CutOrder)
  int64_t n_grid = 0;
  void set_tree(int max_levels);   // dims from rec_n
  // line records [pt_batch][rec_n] (32 B), then with selection the thresholds of the
  // groups of kSelGroup tiles [pt_batch][n_groups()] (8 B), or with the far field by moments
  // the tree [pt_batch][n_nodes] and, when any point goes by tiles, the far sums
  // [pt_batch][n_grid] (8 B) and the near ranges [pt_batch][n_tiles] (16 B), then the lines'
  // bounds [pt_batch] and the orders by cut: moments, then keys
  int64_t n_groups() const { return (n_tiles + kSelGroup - 1) / kSelGroup; }
  size_t tau_offset() const { return (size_t)rec_n * pt_batch * 32; }
  size_t node_offset() const { return tau_offset(); }
  size_t far_offset() const {
    return node_offset() + (size_t)pt_batch * dims.n_nodes * node_bytes(moments);
  }
  size_t near_offset() const {
    return far_offset() + (any_tile ? ((size_t)pt_batch * n_grid * 8 + 15) / 16 * 16 : 0);
  }
  size_t bounds_offset() const {
    return near_offset() + (any_tile ? (size_t)pt_batch * n_tiles * sizeof(NearRange) : 0);
  }
  size_t pre_offset() const {   // (128 B: a row of moments lies in whole cache lines)
    return (bounds_offset() + (size_t)pt_batch * sizeof(PtBounds) + 127) / 128 * 128;
  }
  size_t pre_bytes() const {    // per point
    return (size_t)cut_blocks * (kCutBlock / 16) * moments * sizeof(double);
  }
  size_t keys_offset() const { return pre_offset() + (size_t)pt_batch * pre_bytes(); }
  size_t keys_bytes() const { return (size_t)cut_blocks * kCutBlock * sizeof(uint32_t); }
  // bytes per P-T point beside the records
  size_t extra_bytes() const {
    return moments ? (size_t)dims.n_nodes * node_bytes(moments) + sizeof(PtBounds) +
                         pre_bytes() + keys_bytes() +
                         (any_tile ? (size_t)n_grid * 8 + (size_t)n_tiles * sizeof(NearRange) : 0)
           : select_eps > 0.0 ? (size_t)n_groups() * 8 : 0;
  }
  size_t rec_bytes() const {
    if (moments) return keys_offset() + (size_t)pt_batch * keys_bytes();
    return tau_offset() + (select_eps > 0.0 ? (size_t)pt_batch * n_groups() * 8 : 0);
  }
  size_t part_bytes(size_t n_grid) const {
    return max_split() > 1 ? (size_t)pt_batch * max_split() * n_grid * sizeof(double) : 0;
  }
};

struct Server;  // serving loop (serve.hip)

// HIP event pairs around tile-kernel launches (events are reused across periods).
struct KernelTimer {
  std::vector<hipEvent_t> ev;
  size_t used = 0;
  int record(hipStream_t st);   // records the next event on st
};

}  // namespace xs

struct xs_ctx {
  int device = 0;
  size_t budget = 0;
  std::atomic<size_t> used{0};
  int n_cu = 0;
  size_t lds = 0;
  std::string arch;
  std::mutex mu;
  uint64_t next_handle = 1;
  std::unordered_map<uint64_t, xs::LinesRes*> lines;
  std::unordered_map<uint64_t, xs::GridRes*> grids;
  // scratch of xs_compute / xs_count_evals (single caller thread)
  xs::Scratch pts_buf, part_buf, out_buf, count_buf, rec_buf, order_buf;
  std::vector<int> order_host;           // content of order_buf
  void* pts_pinned = nullptr;
  size_t pts_pinned_cap = 0;
  std::vector<double> pts_host;          // content of pts_buf
  hipEvent_t pts_event = nullptr;        // recorded after the last launch reading scratch
  bool pts_event_valid = false;
  hipStream_t last_stream = nullptr;
  xs::Server* server = nullptr;
  std::mutex serve_mu;                   // guards starting the server
  xs::KernelTimer* timer = nullptr;      // non-null while kernel timing is enabled
  std::set<xs_graph*> graphs;            // live graphs (guarded by mu)
  void* noalloc_scratch = nullptr;       // this device's allocation-free scratch array
  std::string noalloc_error;             // why it is missing (nullptr above)

  bool reserve(size_t bytes);
  void release(size_t bytes);
  int dev_alloc(void** p, size_t bytes, const char* what);
  // dev_alloc, and where the budget is short, again without the scratch that finished calls
  // left (not from the serving calls: the scratch belongs to the context's own thread)
  int dev_alloc_again(void** p, size_t bytes, const char* what);
  void dev_free(void* p, size_t bytes);
  int scratch(xs::Scratch& s, size_t bytes, const char* what);
  // Gives back the scratch of finished calls (all but the point table), after the last launch
  // that reads it.
  void drop_scratch();
  xs::LinesRes* find_lines(xs_lines_t h);
  xs::GridRes* find_grid(xs_grid_t h);
};

namespace xs {
using Ctx = xs_ctx;

extern thread_local std::string g_last_error;   // message of this thread's last failure
int fail(int code, const char* fmt, ...);
int hip_fail(hipError_t e, const char* what);
int validate_opts(const xs_opts* o);
int validate_pts(const xs_pt* pts, size_t npts);
// Launch plan; cap_bytes bounds the records and partials of one batch of (P, T) points
// (0: min(64 GiB, a third of the free budget)); max_item_lines > 0 caps the line range
// of a work item when the split is automatic. The launch shape (P, split) depends only on
// the inputs, the options, max_item_lines and far_moments, never on the memory left (which only
// bounds the points per batch; a caller short of memory asks again with far_moments false).
// items_per_slot > 0 sets the work items per resident wavefront slot of the automatic
// split (default 4). With pts_per_lane, split and waves_per_simd all 0 the shape comes
// from the tuning cache when it holds the workload's class. far_moments false: every line by
// the tile kernel (the callers' second choice where memory for the moments is missing).
Plan make_plan(Ctx& c, const LinesRes& L, const GridRes& G, const xs_pt* pts, size_t npts,
               const xs_opts& o, size_t cap_bytes = 0, int64_t max_item_lines = 0, int items_per_slot = 0,
               bool far_moments = true);

// Lines [lo, hi) that can reach [first, last] within cut (from the sampled index; the
// range errs on the inclusive side).
void line_range_nu(const LinesRes& L, double first, double last, double cut, int64_t* lo,
                   int64_t* hi);
int upload_pts(Ctx& c, const xs_pt* pts, size_t npts, hipStream_t st);

// Tuning cache (tune.hip): launch shapes per workload class, process-wide.
// Occupancy target of the tile kernel for the option value w (0 automatic, 2 the
// compiler's own choice, 3..6 waves per SIMD); the returned 0 means no target. The
// automatic value is 5 on the FP32 path with up to 2 points per lane (measured fastest
// untuned on the mid and table workloads: 96 VGPRs with few spills; 6 waves cap the
// kernel at 80 VGPRs and spill in the far-line code) and the compiler's choice otherwise.
inline int waves_target(int w, int P, bool f64) {
  if (w == 0) return (!f64 && P <= 2) ? 5 : 0;
  return w == 2 ? 0 : w;
}
// The option value of a target (2 for none).
inline int waves_option(int target) { return target == 0 ? 2 : target; }

// A cached launch shape; W is an option value (2..6).
struct TuneVal {
  int P = 2, W = 5, ips = 4;
  double probe_ms = 0.0;
};
std::string tune_key(const Ctx& c, const LinesRes& L, const GridRes& G, size_t npts,
                     const xs_opts& o);
bool tune_get(const std::string& key, TuneVal* v);
void tune_put(const std::string& key, const TuneVal& v);
// Enqueue the whole path on `st`: per batch of (P, T) points the parameter kernel, the
// tile kernel and (split > 1) the fixed-order reduction; with counts != nullptr the count
// kernel instead of tile + reduction. out_dev holds rows of o.out_dtype elements.
int enqueue_path(const LinesRes& L, const GridRes& G, const xs_opts& o, const Plan& p,
                 const double* pts_dev, const int* order_dev, void* out_dev, void* rec_dev,
                 void* part_dev, hipStream_t st, unsigned long long* counts = nullptr,
                 KernelTimer* tm = nullptr);
// One step of the path for the batch of points [pt0, pt0 + nb): the parameter kernel
// (with_params), the tile kernel over positions [c0, c1) of the tile order (order_dev is
// required), and the fixed-order reduction of the batch (with_reduce, split > 1). The
// steps of one batch must run in this order.
int enqueue_step(const LinesRes& L, const GridRes& G, const xs_opts& o, const Plan& p,
                 const double* pts_dev, const int* order_dev, void* out_dev, void* rec_dev,
                 void* part_dev, hipStream_t st, int pt0, int nb, int64_t c0, int64_t c1,
                 bool with_params, bool with_reduce, unsigned long long* counts = nullptr,
                 KernelTimer* tm = nullptr);
// Upload the plan's tile order into the context buffer (skipped when unchanged).
int upload_order(Ctx& c, const Plan& p, hipStream_t st);

// Bytes of one sigma element for the output type of the options.
inline size_t out_elem_bytes(const xs_opts& o) {
  return o.out_dtype == XS_F32 ? sizeof(float) : sizeof(double);
}

inline void free_lines_res(Ctx& c, LinesRes* L) {
  c.dev_free(L->base, L->bytes);
  delete L;
}

void serve_shutdown(Ctx* c);
// Release the device resources of every graph of the context (xs_destroy).
void graphs_release_all(Ctx* c);

}  // namespace xs
