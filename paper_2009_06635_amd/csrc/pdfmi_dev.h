// Device-side data layout shared by the host runtime (pdfmi.cpp) and the
// kernels (kernels.hip).  Not part of the public ABI.
#pragma once
#include <stdint.h>

#include <map>
#include <mutex>
#include <utility>

#include <hip/hip_runtime.h>

namespace pdfmi {

constexpr int kMaxSub = 16;      // Q^2 sub-grids per member
constexpr int kMaxReq = 64;      // flavours per query call
constexpr int kMaxSeg = 16;      // alpha_s segments

// Region / mode bits of a query point.
enum : int { kLowX = 1, kLowQ = 2, kHighQ = 4, kInvalid = 8, kXHigh = 16 };

// Per-cell Hermite data of one 1D knot table (cell i = [t_i, t_{i+1}]), FP64,
// computed on the host.  With Hermite basis h00,h10,h01,h11 of the cell
// parameter u, hl = Delta_i / (2 Delta_{i-1}) and hr = Delta_i / (2 Delta_{i+1}),
// the weights of the four knots i-1..i+2 are
//   w(-1) = -hl h10                           w(1) = h01 + el h10 + (er - hr) h11
//   w(0)  = h00 + (hl - el) h10 - er h11      w(2) = hr h11
// (finite-difference slopes: the mean of the adjacent secants inside the
// table, where el = er = 1/2; the one secant at its ends: at the first cell
// hl = 0 and el = 1, at the last hr = 0 and er = 1).  48 bytes: three 16-byte
// LDS reads per cell.
struct alignas(16) CellCoef {
  double t0;      // knot i
  double inv_t0;  // 1 / knot i
  double invD;    // 1 / ln(knot i+1 / knot i)
  double hl, hr;  // half ratios of the neighbouring cells' log-widths, 0 at a table end
  float el, er;   // 1/2, or 1 at a table end
};

// A Q^2 cell of any sub-grid: the cells of all sub-grids form one table in
// increasing Q^2 (a threshold's knot starts the upper sub-grid's first cell),
// so one search finds sub-grid and cell together.  80 bytes: an odd number of
// 16-byte units, so that random cells spread over all LDS banks.
struct alignas(16) QCell {
  CellCoef c;
  int row;   // grid row (of P values) of this cell's first stencil Q^2 knot at x knot 0
  int nqp;   // rows between consecutive x knots
  int kiq;   // sub-grid << 16 | cell within the sub-grid
  int d;     // position of the cell's knot i in the stencil: 0 left end, 1 inside, 2 right end
  int pad[4];
};

// An alpha_s cell: value at its first knot, difference to the second, and the
// slopes at both times the cell's log-width (the table's values are fixed, so
// the finite differences are formed once).  80 bytes, as QCell.
struct alignas(16) AsCell {
  double t0, inv_t0, invD;
  double f0, df, d0, d1;
  double pad[3];
};

// Entry i of the logarithm's table (see fast_log): inv = 1 / c_i, log = ln c_i.
struct alignas(16) LogEntry {
  double inv, log;
};
constexpr int kLogEntries = 128;
constexpr int kLogOrigin = 0x3fe60000;  // high word of 0.6875, the smallest reduced argument

// Knot search by bucket hints: positive doubles order like their IEEE-754
// bit patterns, so the key (high word >> shift) of a query selects a bucket of
// a 1D knot table; the bucket's hint is the largest cell index whose knot is
// <= the bucket's smallest value, and at most two more knots lie inside any
// bucket.  The cell of v is then the hint advanced over the next two knots
// that are <= v -- the same index as a binary search with the same raw FP64
// comparisons.  A table with no hint list (off < 0) is binary searched.
struct HintAxis {
  int off;    // first hint in the table block's hints, -1 for none
  int n;      // buckets
  int shift;  // key = high word(v) >> shift
  int key0;   // key of the first knot
};

// x axis of a sub-grid (used when the sub-grids' x knots differ).
struct SubDesc {
  int nx;
  int xk_off, xc_off;  // knot and cell offsets into the table block's knots and cells
  HintAxis xh;
};

// The point-location tables of a member are one contiguous device block of
// tbl_bytes -- knots (x tables, then the Q^2 knots of all sub-grids, thresholds
// once), x cells, Q^2 cells, search hints, sub-grid x axes, logarithm table --
// copied whole into LDS by the kernels when it fits there.  The grid values
// are rows of P columns, row (k, ix, iq) at row_off_k + ix nqp_k + iq.
struct MemberDev {
  int K;                 // sub-grids
  int P;                 // stored columns
  int P64, P32;          // row strides of v64 / v32 (zero padding; FP64 rows are whole 64/128-byte lines)
  int rows;              // rows of all sub-grids
  int64_t elems64, elems32;  // value elements (padded) of v64 / v32
  int tbl_bytes;         // bytes of the location-table block (multiple of 16)
  int cells_off, qcells_off, hints_off, subs_off, logt_off;  // byte offsets in it
  int nqk, qk_off;       // Q^2 knots of all sub-grids, their offset in the knots
  HintAxis qh;
  int shared_x;          // every sub-grid has sub-grid 0's x knots: the axis below
  int nx, xk_off, xc_off;
  HintAxis xh;
  double xmin, xmax;     // x range (shared by all sub-grids)
  double qmin, qmax;     // Q^2 range (first knot of sub-grid 0, last of K-1)
  const unsigned char* tables;  // device, the location-table block
  const double* v64;     // device, FP64 values
  const float* v32;      // device, FP32-rounded values
};

struct ReqCols {
  int n;                     // requested flavours
  signed char col[kMaxReq];  // stored column (< 64), or -1 for a valid flavour absent from the grid
};

struct LaunchCfg {
  int n_cu;           // compute units
  int blocks_per_cu;  // workgroups per CU for the global-grid kernels
  int vector_cols;    // use G-wide column groups for all-column requests
};

// alpha_s table: the cells of all segments in increasing Q^2, one contiguous
// device block -- knots [ncell + 1] (thresholds once, padded to an even
// count), cells, hints, logarithm table -- of `bytes` bytes.
struct AlphasDev {
  int ncell;
  int bytes;               // whole block (multiple of 16); the logarithm table is its tail
  int cells_off, hints_off, logt_off;
  HintAxis h;
  double q_lo, q_hi;       // first and last knot
  double a_lo, a_hi;       // constant values below and above
  const unsigned char* tables;  // device
};

}  // namespace pdfmi

namespace pdfmi {

constexpr int kCompactCols = 12;  // columns of a compacted row (FP32, LDS) of a batched plan

// One request of a batched plan (device copy).
struct BatchReq {
  int member;        // index into the plan's member table
  int R;             // requested flavours
  int col_off;       // offset in the plan's column array of its column list [R], then the output position of
                     // each stored column (-1: not requested) when layout >= 0
  int layout;        // number of its (member, column list) among the plan's, or -1 if not staged compacted
  int all_cols;      // 1 if the request is every stored column in load order
  const double* x;
  const double* q2;
  void* out;         // FP32 or FP64 point-major [n][R], per the plan
  int64_t n;
};

// A tile: tile_points consecutive points of one request (the last tile of a
// request may be shorter).
struct BatchTile {
  int req;
  int count;
  int64_t start;
};

// What a batched run in flight has to itself: how many tiles after each
// workgroup's first have been taken, and how many workgroups have left.  Both
// are 0 between runs (the last workgroup to leave clears them).
struct alignas(64) RunSlot {
  unsigned taken, left;
};

// A compacted copy of a member's FP64 values that a plan makes (device copy).
struct CompactJob {
  const double* src;
  double* dst;
  int64_t elems;  // values of the copy
  int Ps, Rp;     // row strides of src and dst
  ReqCols rc;
};

// Kernel node parameters of one batched run (the persistent kernel).
struct BatchLaunch {
  const void* main_fn;
  unsigned grid, block;
  size_t shm;
  bool counted;  // more tiles than workgroups: the run takes tiles from a RunSlot
};

// Surrogate input normalisation and output envelope (device tables).  The
// envelope of column c is a signed cubic Hermite in ln x through one value
// per sub-grid-0 x knot (the grid value of largest magnitude over every Q^2
// knot at that x), with finite-difference slopes (mean of the adjacent
// secants, the one secant at the ends).
struct SurDev {
  int P;              // stored columns (<= 16)
  int nx;             // envelope knots (sub-grid 0 x knots)
  double lx0, ilx;    // u = 2 (ln x - lx0) * ilx - 1
  double lq0, ilq;    // v = 2 (ln Q^2 - lq0) * ilq - 1
  const double* lxk;  // [nx] ln of the envelope knots
  const float* env;   // [nx][16] envelope values
  const float* envd;  // [nx][16] envelope slopes d E / d ln x
  // inference trusts the network inside sub-grid k for txlo[k] <= x < txhi[k]
  // and tqlo[k] <= Q^2 < tqhi[k] (second to second-last knots) when trust[k]
  int K;
  double qfirst[kMaxSub];  // first Q^2 knot of each sub-grid
  int trust[kMaxSub];
  double txlo[kMaxSub], txhi[kMaxSub], tqlo[kMaxSub], tqhi[kMaxSub];
};

// Device-side state of a surrogate's training call.  The training kernels
// read the global step (which batch slice, which learning rate) from here,
// so every step is the same launch sequence and can be replayed as a graph.
struct SurStep {
  int64_t step;      // global step: batch (step % nb), learning rate, Adam update number step + 1
  int64_t call;      // step index within the current train call (index into loss_out)
  int64_t nb;        // batches in the training set
  int64_t row;       // first row of this step's batch: (step % nb) * batch
  int total;         // cosine schedule length
  float lr0, lrf;    // schedule end points
  float* loss_out;   // the call's per-step losses, or null
  float lr, c1, c2;  // this step's learning rate and bias corrections (written by k_train_fb, read by k_train_update)
};

// Surrogate device buffers (parameters, Adam moments, gradient, training workspace).
// Matrix operands are BF16 pairs (hi, lo) with value = hi + lo.
struct SurBufs {
  float* P;                 // FP32 master parameters
  unsigned short* Pb;       // BF16 halves of the parameters: [0, n) hi, [n, 2n) lo, then the transposed hi halves
  float *M, *V, *G;         // Adam moments, gradient
  float* loss;              // [1]
  float* wpart;             // per-slice partial gradients and losses of a training step
  SurStep* st;              // training-call state
};

// hipFuncSetAttribute(MaxDynamicSharedMemorySize) only when a launch needs
// more dynamic LDS than the kernel was last allowed on this device: repeated
// launches of the same shape make no extra runtime call (it costs several
// microseconds, the whole duration of a small evaluation).
inline hipError_t allow_dynamic_lds(const void* fn, size_t bytes) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, size_t> allowed;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  size_t& a = allowed[{fn, dev}];
  if (bytes <= a) return hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) a = bytes;
  return e;
}

}  // namespace pdfmi
