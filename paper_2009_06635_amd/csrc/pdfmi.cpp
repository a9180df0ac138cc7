// Host runtime of libpdfmi.so: argument and grid validation, member registry,
// per-cell Hermite coefficients, device packing/upload, flavour->column tables,
// error state and kernel launches.  Implements include/pdfmi.h.
#include "pdfmi.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cerrno>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "layouts.h"
#include "pdfmi_dev.h"
#include "tiles.h"

namespace pdfmi {
size_t xfxq2_shared_bytes(const MemberDev& m, bool f32, bool small);
size_t alphas_lds_bytes(const AlphasDev* A, bool member_tables);
hipError_t launch_xfxq2_f64(const MemberDev&, const ReqCols&, const double*, const double*, int64_t, double*,
                            unsigned long long*, int, double, const LaunchCfg&, const AlphasDev*, double*, bool,
                            hipStream_t);
hipError_t launch_compact(const MemberDev& m, const ReqCols& rc, bool f32, int Rp, void* dst, hipStream_t s);
hipError_t launch_compact_jobs(const CompactJob* jobs, int n, int64_t max_elems, hipStream_t s);
hipError_t launch_xfxq2_f32(const MemberDev&, const ReqCols&, const double*, const double*, int64_t, float*,
                            unsigned long long*, int, double, const LaunchCfg&, const AlphasDev*, double*, bool,
                            hipStream_t);
hipError_t launch_locate(const MemberDev&, const double*, const double*, int64_t, int32_t*, int32_t*, int32_t*,
                         int8_t*, int, hipStream_t);
hipError_t launch_alphas(const AlphasDev&, const double*, int64_t, double*, unsigned long long*, int, hipStream_t);
int64_t mc_partials(int64_t n);
size_t batch_shared_bytes(int max_tbl, bool f32, bool lds, int block);
BatchLaunch batch_launch_params(bool f32, bool lds, int max_tbl, int64_t max_elems, int n_cu, int ntiles, int block);
hipError_t batch_prepare(const BatchLaunch& L);
hipError_t batch_launch(const BatchLaunch& L, void** args, hipStream_t s);
int sur_nparams();
int sur_halves();
constexpr int kSurMaxEnvKnots = 512;   // the inference kernel stages the envelope in LDS
constexpr int kAlphasMaxHints = 2048;  // alpha_s search hints staged in LDS
int sur_out_width();
int sur_hidden();
int sur_slices(int B);
size_t sur_workspace_floats(int B);
hipError_t sur_train_prepare();
hipError_t sur_forward_backward(const SurBufs& b, const float* in, const float* T, int B, float* loss_out,
                                hipStream_t s);
hipError_t sur_train_begin(const SurBufs& b, int64_t step, int64_t nbatches, int B, int total, float lr0, float lrf,
                           float* loss_out, hipStream_t s);
hipError_t sur_train_step(const SurBufs& b, const float* in, const float* T, int B, hipStream_t s);
hipError_t sur_adam(const SurBufs& b, float lr, int step, hipStream_t s);
hipError_t sur_refresh_bf16(const SurBufs& b, hipStream_t s);
hipError_t sur_prep(const SurDev& S, const MemberDev& m, const double* x, const double* q2, const double* xf,
                    int64_t n, float* in, float* T, unsigned char* keep, hipStream_t s);
hipError_t sur_gather(const float* in_all, const float* T_all, const int64_t* idx, int64_t n, float* in, float* T,
                      hipStream_t s);
hipError_t sur_infer(const SurDev& S, const MemberDev& m, const ReqCols& rc, const SurBufs& b, const double* x,
                     const double* q2, int64_t n, float* out, double invL01, unsigned long long* nerr, int n_cu,
                     hipStream_t s);
template <typename T>
hipError_t launch_mc_sum(const T*, const T*, int, const double*, int64_t, double*, double*, hipStream_t);
template <typename T>
hipError_t launch_mc_fused(const MemberDev&, const ReqCols&, const AlphasDev&, const double*, const double*,
                           const double*, int64_t, double*, double*, unsigned long long*, double, int, hipStream_t);
hipError_t launch_fk_contract(const double* F, const double* FK, int nrep, int ndat, int64_t K, double* T, int S,
                              double* ws, hipStream_t s);
int fk_slices(int nrep, int ndat, int64_t K, int n_cu);
int fk_limit_slices(int nrep, int ndat, int64_t K, int n_cu);
size_t fk_scratch_bytes();
hipError_t fk_scratch_setup(int device, double** out);
}  // namespace pdfmi

using namespace pdfmi;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int fail_hip(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? PDF_ERR_NOMEM : PDF_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace

namespace pdfmi {
// Error reporting for the library's other host sources (same thread-local message).
int report_error(int code, const char* msg) { return fail(code, "%s", msg); }
}  // namespace pdfmi

namespace {

// A copy of a member's values that holds the columns of one request, in request order.
struct Layout {
  LayoutKey key;
  int stride = 0;        // values per row
  void* mem = nullptr;
  hipEvent_t filled = nullptr;  // recorded after the copy on the stream that made it
  bool ready = false;    // the event has been seen complete
};

void layout_release(Layout& l) {
  if (l.filled) (void)hipEventDestroy(l.filled);
  if (l.mem) (void)hipFree(l.mem);
  l.filled = nullptr;
  l.mem = nullptr;
  l.ready = false;
}

struct Member {
  bool used = false;
  std::vector<Layout> layouts;  // at most kMaxLayouts
  LayoutsWanted wanted;
  MemberDev dev{};
  void* dmem = nullptr;
  std::vector<int> pids;   // stored column -> pid (0 normalised to 21)
  std::vector<int> h_shape;       // host copy of the load arguments (surrogate envelopes)
  std::vector<double> h_knots, h_values;
  double invL01 = 0.0;
  uint64_t gen = 0;        // load generation: a slot reused by a later load gets a new one
  size_t mc_bytes = 0;     // the member's share of the table size that pdf_mc_fused accepts
};

std::mutex g_mu;
std::vector<Member> g_members;
uint64_t g_load_gen = 0;
bool g_init = false;
int g_ncu = 0;
std::string g_arch;  // device architecture name (autotune cache keys)
unsigned long long* g_nerr = nullptr;
bool g_has_alphas = false;
AlphasDev g_alphas{};
size_t g_alphas_mc_bytes = 0;  // the alpha_s table's share of the table size that pdf_mc_fused accepts
void* g_alphas_mem = nullptr;
int g_lds_policy = 0;  // 0 auto, 1 never stage the grid in LDS, 2 whenever it fits
int g_vector_cols = 1; // serve all-column requests with G-wide vector gathers
int g_blocks_per_cu = 32;
void* g_fk_ws = nullptr;      // partial sums of the K slices of pdf_fk_contract (grow-only)
size_t g_fk_ws_bytes = 0;
double* g_fk_scratch = nullptr;  // device address of the fixed scratch of pdf_fk_contract_noalloc
constexpr size_t kLdsBytes = 160 * 1024;

// The part of the set-up that allocates nothing: the device, its compute
// units and the device address of the fixed FK scratch array.
bool g_dev_ready = false;
int ensure_device() {
  if (g_dev_ready) return PDF_OK;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  e = hipDeviceGetAttribute(&g_ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDeviceProperties");
  g_arch = prop.gcnArchName;
  for (char& c : g_arch)
    if (c == ' ' || c == '\t') c = '_';
  e = fk_scratch_setup(dev, &g_fk_scratch);
  if (e != hipSuccess) return fail_hip(e, "hipGetSymbolAddress(fk scratch)");
  g_dev_ready = true;
  return PDF_OK;
}

int ensure_init() {
  if (g_init) return PDF_OK;
  int rc = ensure_device();
  if (rc != PDF_OK) return rc;
  hipError_t e = hipMalloc(&g_nerr, sizeof(unsigned long long));
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(error counter)");
  e = hipMemset(g_nerr, 0, sizeof(unsigned long long));
  if (e != hipSuccess) return fail_hip(e, "hipMemset(error counter)");
  g_init = true;
  return PDF_OK;
}

bool valid_pid(int p) { return (p >= -6 && p <= 6) || p == 21; }
int norm_pid(int p) { return p == 0 ? 21 : p; }

// Hermite coefficients of every cell of a strictly increasing 1D table
// (see CellCoef).
void cell_coefs(const double* t, int n, CellCoef* out) {
  std::vector<double> D(n - 1);
  for (int i = 0; i + 1 < n; ++i) D[i] = std::log(t[i + 1] / t[i]);
  for (int i = 0; i + 1 < n; ++i) {
    CellCoef c{};
    c.t0 = t[i];
    c.inv_t0 = 1.0 / t[i];
    c.invD = 1.0 / D[i];
    const bool L = i > 0, R = i + 1 < n - 1;
    c.hl = L ? 0.5 * (D[i] / D[i - 1]) : 0.0;
    c.hr = R ? 0.5 * (D[i] / D[i + 1]) : 0.0;
    c.el = L ? 0.5f : 1.0f;
    c.er = R ? 0.5f : 1.0f;
    out[i] = c;
  }
}

bool strictly_increasing(const double* t, int n) {
  for (int i = 0; i < n; ++i)
    if (!std::isfinite(t[i])) return false;
  for (int i = 0; i + 1 < n; ++i)
    if (!(t[i] < t[i + 1])) return false;
  return true;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Bucket hints of a strictly increasing table of positive knots (HintAxis):
// the coarsest buckets (largest shift) with at most two knots strictly
// inside any of them, provided the list stays within kMaxHintsPerAxis;
// otherwise no list (the kernels binary search that table).
constexpr int kMaxHintsPerAxis = 4096;

uint64_t double_bits(double v) {
  uint64_t u;
  std::memcpy(&u, &v, 8);
  return u;
}

// The buckets of a table's hint list (off stays -1); n == 0 if it has none.
HintAxis hint_buckets(const double* t, int n) {
  HintAxis h{-1, 0, 0, 0};
  if (n < 4) return h;
  std::vector<int> inside;
  for (int shift = 52; shift >= 32; --shift) {
    const uint64_t k0 = double_bits(t[0]) >> shift, k1 = double_bits(t[n - 1]) >> shift;
    const uint64_t nb = k1 - k0 + 1;
    if (nb > (uint64_t)kMaxHintsPerAxis) break;  // finer buckets only make the list longer
    inside.assign(nb, 0);
    const uint64_t low_mask = (1ull << shift) - 1;
    for (int i = 0; i < n; ++i) {
      const uint64_t u = double_bits(t[i]);
      if (u & low_mask) ++inside[(u >> shift) - k0];  // above the bucket's smallest value
    }
    if (*std::max_element(inside.begin(), inside.end()) > 2) continue;
    h.n = (int)nb;
    h.shift = shift - 32;
    h.key0 = (int)k0;
    break;
  }
  return h;
}

HintAxis build_hints(const double* t, int n, std::vector<short>& hints) {
  HintAxis h = hint_buckets(t, n);
  if (h.n == 0) return h;
  h.off = (int)hints.size();
  for (int b = 0; b < h.n; ++b) {
    const uint64_t lo_bits = (uint64_t)(h.key0 + b) << (h.shift + 32);
    double lo;
    std::memcpy(&lo, &lo_bits, 8);
    const int i = (int)(std::upper_bound(t, t + n, lo) - t) - 1;  // largest i with t[i] <= lo
    hints.push_back((short)std::min(std::max(i, 0), n - 2));
  }
  return h;
}

// Table of fast_log: interval i of [0.6875, 1.375) (width 2^-8 below 1, 2^-7
// above); inv the one of 64 candidates near 1 / its middle whose -ln is
// nearest to a double, 1 next to 1.
std::vector<LogEntry> make_log_table() {
  std::vector<LogEntry> t(kLogEntries);
  for (int i = 0; i < kLogEntries; ++i) {
    // interval i starts at the double with high word kLogOrigin + (i << 13)
    auto start = [](int j) {
      const uint64_t u = (uint64_t)(uint32_t)(kLogOrigin + (j << 13)) << 32;
      double v;
      std::memcpy(&v, &u, 8);
      return v;
    };
    const double a = start(i), b = start(i + 1);
    t[i] = LogEntry{1.0, 0.0};
    if (a == 1.0 || b == 1.0) continue;
    long double best = 1.0L;
    for (int j = -32; j < 32; ++j) {
      const double inv = 2.0 / (a + b) * (1.0 + j * 0x1p-20);
      const long double l = -std::log((long double)inv);
      const long double err = std::fabs((l - (long double)(double)l) / l);
      if (err < best) {
        best = err;
        t[i] = LogEntry{inv, (double)l};
      }
    }
  }
  return t;
}
const std::vector<LogEntry>& log_table() {
  static const std::vector<LogEntry> t = make_log_table();
  return t;
}

int check_stream_args(const void* a, const void* b, int64_t n) {
  if (n < 0) return fail(PDF_ERR_ARG, "n < 0");
  if (n > 0 && (!a || !b)) return fail(PDF_ERR_ARG, "null device pointer");
  return PDF_OK;
}

int build_req(const Member& M, const int32_t* pids, int32_t n_pids, ReqCols& rc) {
  if (!pids) {
    if ((int)M.pids.size() > kMaxReq) return fail(PDF_ERR_ARG, "too many stored flavours for one call");
    rc.n = (int)M.pids.size();
    for (int j = 0; j < rc.n; ++j) rc.col[j] = j;
    return PDF_OK;
  }
  if (n_pids < 1 || n_pids > kMaxReq) return fail(PDF_ERR_ARG, "n_pids must be in [1, %d]", kMaxReq);
  rc.n = n_pids;
  for (int j = 0; j < n_pids; ++j) {
    if (!valid_pid(pids[j])) return fail(PDF_ERR_PID, "invalid flavour id %d", pids[j]);
    const int p = norm_pid(pids[j]);
    rc.col[j] = -1;
    for (size_t c = 0; c < M.pids.size(); ++c)
      if (M.pids[c] == p) rc.col[j] = (int)c;
  }
  return PDF_OK;
}

Member* get_member(int32_t id) {
  if (id < 0 || id >= (int32_t)g_members.size() || !g_members[id].used) return nullptr;
  return &g_members[id];
}

// Stage the whole grid in LDS for this call?
// extra: further LDS bytes the launch needs (the alpha_s table of a fused call).
int lds_grid_elems(const MemberDev& dev, bool f32, int64_t n, size_t extra = 0) {
  if (g_lds_policy == 1) return 0;
  const int64_t elems = f32 ? dev.elems32 : dev.elems64;
  const size_t values = (size_t)elems * (f32 ? 4 : 8) + extra;
  const bool small = values + xfxq2_shared_bytes(dev, f32, false) > kLdsBytes - 1024;
  const size_t bytes = values + xfxq2_shared_bytes(dev, f32, small);
  if (bytes > kLdsBytes - 1024) return 0;
  if (g_lds_policy == 0) {
    // each workgroup pays one grid copy; require enough tiles to amortise it,
    // more of them for the smaller workgroup, which gains less (FP64 with
    // alpha_s, 20 x 22 x 13 values, 3e5 and 2e6 points: 32 and 112 us, from
    // global memory 31 and 135; 50 x 36 x 4, 1.1e6 points: 36.4 and 34.2)
    const int64_t tiles = (n + 255) / 256;
    const int per_cu = (int)(kLdsBytes / bytes);
    const int least = !small ? 4 : (dev.P > 8 ? 10 : 24);
    if (tiles < (int64_t)least * g_ncu * (per_cu > 0 ? per_cu : 1)) return 0;
  }
  return (int)elems;
}

}  // namespace

// ---------------------------------------------------------------------------------------

extern "C" int pdf_validate_grid(int32_t K, const int32_t* shape, int32_t P, const int32_t* pids,
                                 const double* knots, const double* values) {
  if (!shape || !pids || !knots || !values) return fail(PDF_ERR_ARG, "null pointer");
  if (K < 1 || K > kMaxSub) return fail(PDF_ERR_GRID, "n_subgrids must be in [1, %d]", kMaxSub);
  if (P < 1 || P > 64) return fail(PDF_ERR_GRID, "n_pids must be in [1, 64]");
  for (int c = 0; c < P; ++c) {
    if (!valid_pid(pids[c])) return fail(PDF_ERR_PID, "invalid stored flavour id %d", pids[c]);
    for (int d = 0; d < c; ++d)
      if (norm_pid(pids[d]) == norm_pid(pids[c])) return fail(PDF_ERR_PID, "duplicated flavour id %d", pids[c]);
  }
  int64_t ko = 0, vo = 0;
  double x0 = 0, x1 = 0, qprev = 0;
  for (int k = 0; k < K; ++k) {
    const int nx = shape[2 * k], nq = shape[2 * k + 1];
    if (nx < 2 || nq < 2 || nx > (1 << 20) || nq > (1 << 20))
      return fail(PDF_ERR_GRID, "sub-grid %d: need nx >= 2 and nq >= 2", k);
    const double* xk = knots + ko;
    const double* qk = knots + ko + nx;
    if (!strictly_increasing(xk, nx) || !(xk[0] > 0.0) || !(xk[nx - 1] <= 1.0))
      return fail(PDF_ERR_GRID, "sub-grid %d: x knots must be strictly increasing in (0, 1]", k);
    if (!strictly_increasing(qk, nq) || !(qk[0] > 0.0))
      return fail(PDF_ERR_GRID, "sub-grid %d: Q^2 knots must be strictly increasing and > 0", k);
    if (k == 0) {
      x0 = xk[0];
      x1 = xk[nx - 1];
    } else {
      if (xk[0] != x0 || xk[nx - 1] != x1) return fail(PDF_ERR_GRID, "sub-grid %d: x range differs from sub-grid 0", k);
      if (qk[0] != qprev) return fail(PDF_ERR_GRID, "sub-grid %d: first Q^2 knot must repeat the previous last knot", k);
    }
    qprev = qk[nq - 1];
    const int64_t nv = (int64_t)nx * nq * P;
    for (int64_t i = 0; i < nv; ++i)
      if (!std::isfinite(values[vo + i])) return fail(PDF_ERR_GRID, "sub-grid %d: non-finite value", k);
    ko += nx + nq;
    vo += nv;
  }
  // the kernels address a member's padded FP64 values with 32-bit byte offsets
  int64_t padded_bytes = 0;
  for (int k = 0; k < K; ++k)
    padded_bytes += (int64_t)std::max(shape[2 * k], 4) * std::max(shape[2 * k + 1], 4) * ((P + 15) & ~15) * 8;
  if (padded_bytes > INT32_MAX) return fail(PDF_ERR_GRID, "grid values exceed 2 GiB");
  if (ko > 8192) return fail(PDF_ERR_GRID, "more than 8192 knots in total (they are staged in LDS)");
  return PDF_OK;
}

extern "C" int pdf_load_grid(int32_t K, const int32_t* shape, int32_t P, const int32_t* pids, const double* knots,
                             const double* values, int32_t* member_out) {
  if (!member_out) return fail(PDF_ERR_ARG, "null member_out");
  int rc = pdf_validate_grid(K, shape, P, pids, knots, values);
  if (rc != PDF_OK) return rc;
  std::lock_guard<std::mutex> lock(g_mu);
  if ((rc = ensure_init()) != PDF_OK) return rc;

  Member M;
  M.used = true;
  for (int c = 0; c < P; ++c) M.pids.push_back(norm_pid(pids[c]));
  {
    int64_t nk = 0, nv = 0;
    for (int k = 0; k < K; ++k) {
      nk += shape[2 * k] + shape[2 * k + 1];
      nv += (int64_t)shape[2 * k] * shape[2 * k + 1] * P;
    }
    M.h_shape.assign(shape, shape + 2 * K);
    M.h_knots.assign(knots, knots + nk);
    M.h_values.assign(values, values + nv);
  }
  MemberDev& d = M.dev;
  d.K = K;
  d.P = P;
  // FP64 rows are whole 64- or 128-byte lines (fewer cache lines per
  // stencil), FP32 rows a multiple of 16 bytes
  const int P64 = P <= 4 ? 4 : (P <= 8 ? 8 : (P + 15) & ~15), P32 = (P + 3) & ~3;
  d.P64 = P64;
  d.P32 = P32;
  // rows of the values: sub-grids with fewer than 4 knots on an axis are padded to 4
  std::vector<int> row_off(K), nqp(K);
  int64_t rows = 0;
  for (int k = 0; k < K; ++k) {
    nqp[k] = std::max(shape[2 * k + 1], 4);
    row_off[k] = (int)rows;
    rows += (int64_t)std::max(shape[2 * k], 4) * nqp[k];
  }
  const int64_t n64 = rows * P64, n32 = rows * P32;
  d.rows = (int)rows;
  d.elems64 = n64;
  d.elems32 = n32;
  // location tables: x knots, cells and hints per sub-grid (those whose x
  // knots equal sub-grid 0's share its tables), and one Q^2 table for all
  // sub-grids (the threshold between two is one knot)
  std::vector<double> hk, hq;
  std::vector<CellCoef> hc;
  std::vector<QCell> hqc;
  std::vector<short> hh;
  std::vector<SubDesc> subs(K);
  std::vector<double> hv((size_t)n64, 0.0);
  std::vector<float> hf((size_t)n32, 0.0f);
  int64_t ko = 0, vo = 0;
  size_t ref_knots = 0, ref_cells = 0, ref_hints = 0;
  d.shared_x = 1;
  for (int k = 0; k < K; ++k) {
    SubDesc& S = subs[k];
    const int nx = shape[2 * k], nq = shape[2 * k + 1];
    const double* xk = knots + ko;
    const double* qk = knots + ko + nx;
    if (k > 0 && nx == subs[0].nx && std::memcmp(xk, knots, sizeof(double) * nx) == 0) {
      S = subs[0];
    } else {
      if (k > 0) d.shared_x = 0;
      S.nx = nx;
      S.xk_off = (int)hk.size();
      hk.insert(hk.end(), xk, xk + nx);
      S.xc_off = (int)hc.size();
      hc.resize(hc.size() + nx - 1);
      cell_coefs(xk, nx, &hc[S.xc_off]);
      S.xh = build_hints(xk, nx, hh);
      ref_hints += S.xh.off < 0 ? 0 : S.xh.n;
      ref_knots += nx;
      ref_cells += nx - 1;
    }
    std::vector<CellCoef> qc(nq - 1);
    cell_coefs(qk, nq, qc.data());
    ref_knots += nq;
    ref_cells += nq - 1;
    for (int i = 0; i + 1 < nq; ++i) {
      const int sq = std::min(std::max(i - 1, 0), nqp[k] - 4);
      hq.push_back(qk[i]);
      hqc.push_back(QCell{qc[i], row_off[k] + sq, nqp[k], k << 16 | i, i - sq, {}});
    }
    if (k == K - 1) hq.push_back(qk[nq - 1]);
    if (K > 1) ref_hints += hint_buckets(qk, nq).n;
    for (int ix = 0; ix < nx; ++ix)
      for (int iq = 0; iq < nq; ++iq)
        for (int c = 0; c < P; ++c) {
          const double v = values[vo + ((int64_t)ix * nq + iq) * P + c];
          const int64_t row = row_off[k] + (int64_t)ix * nqp[k] + iq;
          hv[row * P64 + c] = v;
          hf[row * P32 + c] = (float)v;
        }
    ko += nx + nq;
    vo += (int64_t)nx * nq * P;
  }
  d.nx = subs[0].nx;
  d.xk_off = subs[0].xk_off;
  d.xc_off = subs[0].xc_off;
  d.xh = subs[0].xh;
  d.nqk = (int)hq.size();
  d.qk_off = (int)hk.size();
  d.qh = build_hints(hq.data(), d.nqk, hh);
  if (K == 1) ref_hints += d.qh.off < 0 ? 0 : d.qh.n;
  hk.insert(hk.end(), hq.begin(), hq.end());
  d.xmin = knots[0];
  d.xmax = knots[shape[0] - 1];
  d.qmin = hq.front();
  d.qmax = hq.back();
  M.invL01 = hqc[0].c.invD;
  // pdf_mc_fused accepts members whose tables, at 8 bytes a knot, 48 a cell, 2
  // a hint and 88 a sub-grid (thresholds and hints counted per sub-grid), fit LDS
  M.mc_bytes = align_up(ref_knots, 2) * 8 + ref_cells * 48 + align_up(ref_hints * 2, 16) +
               align_up((size_t)K * 88, 16);

  // table block, 16-byte aligned parts
  const std::vector<LogEntry>& lt = log_table();
  d.cells_off = (int)align_up(hk.size() * 8, 16);
  d.qcells_off = d.cells_off + (int)(hc.size() * sizeof(CellCoef));
  d.hints_off = d.qcells_off + (int)(hqc.size() * sizeof(QCell));
  d.subs_off = d.hints_off + (int)align_up(hh.size() * sizeof(short), 16);
  d.logt_off = d.subs_off + (int)align_up((size_t)K * sizeof(SubDesc), 16);
  d.tbl_bytes = d.logt_off + (int)(lt.size() * sizeof(LogEntry));
  const size_t bt = align_up((size_t)d.tbl_bytes, 256);
  const size_t b64 = align_up((size_t)n64 * sizeof(double), 256);
  const size_t b32 = align_up((size_t)n32 * sizeof(float), 256);
  std::vector<unsigned char> blob(bt + b64 + b32, 0);
  std::memcpy(blob.data(), hk.data(), hk.size() * sizeof(double));
  std::memcpy(blob.data() + d.cells_off, hc.data(), hc.size() * sizeof(CellCoef));
  std::memcpy(blob.data() + d.qcells_off, hqc.data(), hqc.size() * sizeof(QCell));
  if (!hh.empty()) std::memcpy(blob.data() + d.hints_off, hh.data(), hh.size() * sizeof(short));
  std::memcpy(blob.data() + d.subs_off, subs.data(), (size_t)K * sizeof(SubDesc));
  std::memcpy(blob.data() + d.logt_off, lt.data(), lt.size() * sizeof(LogEntry));
  std::memcpy(blob.data() + bt, hv.data(), (size_t)n64 * sizeof(double));
  std::memcpy(blob.data() + bt + b64, hf.data(), (size_t)n32 * sizeof(float));

  hipError_t e = hipMalloc(&M.dmem, blob.size());
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(grid)");
  e = hipMemcpy(M.dmem, blob.data(), blob.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(M.dmem);
    return fail_hip(e, "hipMemcpy(grid)");
  }
  unsigned char* base = static_cast<unsigned char*>(M.dmem);
  d.tables = base;
  d.v64 = reinterpret_cast<const double*>(base + bt);
  d.v32 = reinterpret_cast<const float*>(base + bt + b64);

  M.gen = ++g_load_gen;
  for (size_t i = 0; i < g_members.size(); ++i) {
    if (!g_members[i].used) {
      g_members[i] = M;
      *member_out = (int32_t)i;
      return PDF_OK;
    }
  }
  g_members.push_back(M);
  *member_out = (int32_t)(g_members.size() - 1);
  return PDF_OK;
}

extern "C" int pdf_unload(int32_t member) {
  std::lock_guard<std::mutex> lock(g_mu);
  Member* M = get_member(member);
  if (!M) return fail(PDF_ERR_MEMBER, "unknown member %d", member);
  hipError_t e = hipFree(M->dmem);
  for (Layout& l : M->layouts) layout_release(l);
  *M = Member();
  if (e != hipSuccess) return fail_hip(e, "hipFree(grid)");
  return PDF_OK;
}

extern "C" int pdf_validate_alphas(int32_t n, const double* q2k, const double* a) {
  if (!q2k || !a) return fail(PDF_ERR_ARG, "null pointer");
  if (n < 2 || n > 256) return fail(PDF_ERR_GRID, "alpha_s table needs 2..256 knots");
  int seg_len = 1, nseg = 1;
  for (int i = 0; i < n; ++i) {
    if (!std::isfinite(q2k[i]) || !(q2k[i] > 0.0) || !std::isfinite(a[i]))
      return fail(PDF_ERR_GRID, "alpha_s knot %d: need finite Q^2 > 0 and finite value", i);
    if (i == 0) continue;
    if (q2k[i] == q2k[i - 1]) {
      if (seg_len < 2) return fail(PDF_ERR_GRID, "alpha_s segment ending at knot %d has < 2 knots", i);
      if (++nseg > kMaxSeg) return fail(PDF_ERR_GRID, "more than %d alpha_s segments", kMaxSeg);
      seg_len = 1;
    } else if (q2k[i] > q2k[i - 1]) {
      ++seg_len;
    } else {
      return fail(PDF_ERR_GRID, "alpha_s Q^2 knots must be non-decreasing");
    }
  }
  if (seg_len < 2) return fail(PDF_ERR_GRID, "last alpha_s segment has < 2 knots");
  return PDF_OK;
}

extern "C" int pdf_load_alphas(int32_t n, const double* q2k, const double* a) {
  int rc = pdf_validate_alphas(n, q2k, a);
  if (rc != PDF_OK) return rc;
  std::lock_guard<std::mutex> lock(g_mu);
  if ((rc = ensure_init()) != PDF_OK) return rc;
  AlphasDev A{};
  // the cells of every segment with their stencil values, the knots once each
  std::vector<double> hk;
  std::vector<AsCell> hc;
  std::vector<short> hh;
  int ref_hints = 0;
  for (int lo = 0, i = 1; i <= n; ++i) {
    if (i < n && q2k[i] != q2k[i - 1]) continue;
    const int m = i - lo;  // knots lo .. i - 1 form a segment
    std::vector<CellCoef> c(m - 1);
    cell_coefs(q2k + lo, m, c.data());
    for (int j = 0; j + 1 < m; ++j) {
      // slopes times the cell's log-width from the weights of CellCoef
      const double f0 = a[lo + j], f1 = a[lo + j + 1];
      const double fm = j > 0 ? a[lo + j - 1] : f0, fp = j + 2 < m ? a[lo + j + 2] : f1;
      const AsCell ac{c[j].t0, c[j].inv_t0, c[j].invD, f0, f1 - f0, c[j].el * (f1 - f0) + c[j].hl * (f0 - fm),
                      c[j].er * (f1 - f0) + c[j].hr * (fp - f1), {}};
      hk.push_back(q2k[lo + j]);
      hc.push_back(ac);
    }
    // hints counted as per-segment lists for the size that pdf_mc_fused accepts
    const int buckets = hint_buckets(q2k + lo, m).n;
    if (ref_hints + buckets <= kAlphasMaxHints) ref_hints += buckets;
    lo = i;
  }
  hk.push_back(q2k[n - 1]);
  A.ncell = (int)hc.size();
  A.h = build_hints(hk.data(), (int)hk.size(), hh);
  if ((int)hh.size() > kAlphasMaxHints) {  // keep the staged list small: binary search
    hh.clear();
    A.h.off = -1;
  }
  A.q_lo = q2k[0];
  A.q_hi = q2k[n - 1];
  A.a_lo = a[0];
  A.a_hi = a[n - 1];
  const std::vector<LogEntry>& lt = log_table();
  A.cells_off = (int)align_up(hk.size() * 8, 16);
  A.hints_off = A.cells_off + (int)(hc.size() * sizeof(AsCell));
  A.logt_off = A.hints_off + (int)align_up(hh.size() * sizeof(short), 16);
  A.bytes = A.logt_off + (int)(lt.size() * sizeof(LogEntry));
  std::vector<unsigned char> blob((size_t)A.bytes, 0);
  std::memcpy(blob.data(), hk.data(), hk.size() * 8);
  std::memcpy(blob.data() + A.cells_off, hc.data(), hc.size() * sizeof(AsCell));
  if (!hh.empty()) std::memcpy(blob.data() + A.hints_off, hh.data(), hh.size() * sizeof(short));
  std::memcpy(blob.data() + A.logt_off, lt.data(), lt.size() * sizeof(LogEntry));
  void* mem = nullptr;
  hipError_t e = hipMalloc(&mem, blob.size());
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(alpha_s)");
  e = hipMemcpy(mem, blob.data(), blob.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(mem);
    return fail_hip(e, "hipMemcpy(alpha_s)");
  }
  A.tables = static_cast<const unsigned char*>(mem);
  g_alphas_mc_bytes = align_up(n, 2) * (8 + 8 + 48) + align_up((size_t)ref_hints, 8) * 2;
  if (g_alphas_mem) (void)hipFree(g_alphas_mem);
  g_alphas_mem = mem;
  g_alphas = A;
  g_has_alphas = true;
  return PDF_OK;
}

// Compacted layouts: a request for some of the stored flavours, or for all in
// another order, reads whole rows of the grid through L2 for the few columns
// it wants, one lane per (point, flavour).  Once kLayoutPoints points have
// been asked of a member with the same request, its columns are copied once
// into rows of their own (kept with the member, at most kMaxLayouts of them
// and kLayoutBytes each), and later calls of that request walk them in
// 16-byte groups like a request for all columns: fewer lines per point (5 of
// 13 columns in FP64: 9 instead of 16) and fewer, wider loads.  5 flavours at
// 3e6 points of the three-sub-grid set in FP64: 201 us without, 116 us with;
// making the copy takes about 50 us, which a call of two million points
// gains back.  Returns the member to evaluate (m or a copy of it in `alt`
// whose values are the layout's), with rc renumbered.

static bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
  (void)hipGetLastError();  // the default stream while another one records a graph
  return true;
}

// While it lives, this thread's calls that a capture forbids leave captures on
// other streams (this thread's or another's) alone.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool ok = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  ~RelaxedCapture() {
    if (ok) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

// Allocates and fills the layout on the caller's stream, without waiting for it.
static bool make_layout(Layout& l, const Member& M, const ReqCols& rc, hipStream_t stream) {
  const RelaxedCapture relaxed;
  if (!relaxed.ok) return false;
  hipError_t e = hipMalloc(&l.mem, (size_t)M.dev.rows * l.stride * (l.key.f32 ? 4 : 8));
  if (e == hipSuccess) e = hipEventCreateWithFlags(&l.filled, hipEventDisableTiming);
  if (e == hipSuccess) e = launch_compact(M.dev, rc, l.key.f32, l.stride, l.mem, stream);
  if (e == hipSuccess) e = hipEventRecord(l.filled, stream);
  if (e == hipSuccess) return true;
  (void)hipGetLastError();
  layout_release(l);
  return false;
}

// Orders the stream after the filling of the layout: at once when that is
// known to be complete, else by its event (not while recording a graph).
static bool layout_ready(Layout& l, hipStream_t stream) {
  if (l.ready) return true;
  if (capturing(stream)) return false;
  const RelaxedCapture relaxed;
  if (!relaxed.ok) return false;
  const hipError_t e = hipEventQuery(l.filled);
  if (e == hipSuccess) return l.ready = true;
  (void)hipGetLastError();
  if (e == hipErrorNotReady && hipStreamWaitEvent(stream, l.filled, 0) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

static const MemberDev* use_layout(Member& M, bool f32, int64_t n, ReqCols& rc, MemberDev& alt, hipStream_t stream) {
  const MemberDev& d = M.dev;
  bool all = rc.n == d.P;
  for (int j = 0; j < rc.n && all; ++j) all = rc.col[j] == j;
  if (all || !g_vector_cols) return &d;
  static_assert(sizeof(LayoutKey::col) == kMaxReq, "a key holds any request");
  LayoutKey key;
  key.f32 = f32;
  key.n = rc.n;
  std::memcpy(key.col, rc.col, (size_t)rc.n);
  Layout* l = nullptr;
  for (Layout& c : M.layouts)
    if (c.key == key) l = &c;
  if (!l) {
    if (M.layouts.size() >= kMaxLayouts) return &d;
    Layout made;
    made.key = key;
    made.stride = layout_stride(rc.n, f32, d.rows, (int64_t)kLdsBytes - 1024 - (int64_t)xfxq2_shared_bytes(d, f32, false));
    // nothing is made while the stream records a graph
    if (!layout_small(f32, d.rows, made.stride) || !M.wanted.add(key, n) || capturing(stream)) return &d;
    if (!make_layout(made, M, rc, stream)) {
      M.wanted.again(key);
      return &d;
    }
    M.wanted.remove(key);
    M.layouts.push_back(made);
    l = &M.layouts.back();
  }
  if (!layout_ready(*l, stream)) return &d;
  alt = d;
  alt.P = rc.n;
  if (f32) {
    alt.P32 = l->stride;
    alt.elems32 = (int64_t)d.rows * l->stride;
    alt.v32 = static_cast<const float*>(l->mem);
  } else {
    alt.P64 = l->stride;
    alt.elems64 = (int64_t)d.rows * l->stride;
    alt.v64 = static_cast<const double*>(l->mem);
  }
  for (int j = 0; j < rc.n; ++j)
    if (rc.col[j] >= 0) rc.col[j] = (signed char)j;
  return &alt;
}

// aout: alpha_s output of a fused call (nullptr: PDFs only).
template <typename T>
static int xfxq2_impl(int32_t member, const int32_t* pids, int32_t n_pids, const double* x, const double* q2,
                      int64_t n, T* out, double* aout, bool fused, pdf_stream_t stream) {
  int rc = check_stream_args(x, q2, n);
  if (rc != PDF_OK) return rc;
  if (n > 0 && !out) return fail(PDF_ERR_ARG, "null out");
  if (fused && n > 0 && !aout) return fail(PDF_ERR_ARG, "null alphas_out");
  std::lock_guard<std::mutex> lock(g_mu);
  Member* M = get_member(member);
  if (!M) return fail(PDF_ERR_MEMBER, "unknown member %d", member);
  if (fused && !g_has_alphas) return fail(PDF_ERR_STATE, "no alpha_s table loaded");
  ReqCols req{};
  if ((rc = build_req(*M, pids, n_pids, req)) != PDF_OK) return rc;
  if (n == 0) return PDF_OK;
  if (n * (int64_t)req.n > ((int64_t)1 << 40)) return fail(PDF_ERR_ARG, "n too large");
  const bool f32 = sizeof(T) == 4;
  MemberDev alt;
  const MemberDev* dev = use_layout(*M, f32, n, req, alt, (hipStream_t)stream);
  const bool compact = dev == &alt;
  const bool stageable = !compact || layout_stageable(req.n, f32, f32 ? alt.P32 : alt.P64);
  const int lds =
      stageable ? lds_grid_elems(*dev, f32, n, alphas_lds_bytes(fused ? &g_alphas : nullptr, true)) : 0;
  hipError_t e;
  const LaunchCfg cfg{g_ncu, g_blocks_per_cu, g_vector_cols};
  const AlphasDev* A = fused ? &g_alphas : nullptr;
  if constexpr (sizeof(T) == 8)
    e = launch_xfxq2_f64(*dev, req, x, q2, n, out, g_nerr, lds, M->invL01, cfg, A, aout, compact,
                         (hipStream_t)stream);
  else
    e = launch_xfxq2_f32(*dev, req, x, q2, n, out, g_nerr, lds, M->invL01, cfg, A, aout, compact,
                         (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch xfxq2");
  return PDF_OK;
}

extern "C" int pdf_xfxq2(int32_t member, const int32_t* pids, int32_t n_pids, const double* x, const double* q2,
                         int64_t n, double* out, pdf_stream_t stream) {
  return xfxq2_impl<double>(member, pids, n_pids, x, q2, n, out, nullptr, false, stream);
}

extern "C" int pdf_xfxq2_f32(int32_t member, const int32_t* pids, int32_t n_pids, const double* x,
                             const double* q2, int64_t n, float* out, pdf_stream_t stream) {
  return xfxq2_impl<float>(member, pids, n_pids, x, q2, n, out, nullptr, false, stream);
}

extern "C" int pdf_xfxq2_alphas(int32_t member, const int32_t* pids, int32_t n_pids, const double* x,
                                const double* q2, int64_t n, double* out, double* alphas_out, pdf_stream_t stream) {
  return xfxq2_impl<double>(member, pids, n_pids, x, q2, n, out, alphas_out, true, stream);
}

extern "C" int pdf_xfxq2_alphas_f32(int32_t member, const int32_t* pids, int32_t n_pids, const double* x,
                                    const double* q2, int64_t n, float* out, double* alphas_out,
                                    pdf_stream_t stream) {
  return xfxq2_impl<float>(member, pids, n_pids, x, q2, n, out, alphas_out, true, stream);
}

extern "C" int pdf_alphas_q2(const double* q2, int64_t n, double* out, pdf_stream_t stream) {
  int rc = check_stream_args(q2, out, n);
  if (rc != PDF_OK) return rc;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_has_alphas) return fail(PDF_ERR_STATE, "no alpha_s table loaded");
  if (n == 0) return PDF_OK;
  hipError_t e = launch_alphas(g_alphas, q2, n, out, g_nerr, g_ncu, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch alphas");
  return PDF_OK;
}

extern "C" int pdf_locate(int32_t member, const double* x, const double* q2, int64_t n, int32_t* k, int32_t* ix,
                          int32_t* iq, int8_t* region, pdf_stream_t stream) {
  int rc = check_stream_args(x, q2, n);
  if (rc != PDF_OK) return rc;
  if (n > 0 && (!k || !ix || !iq || !region)) return fail(PDF_ERR_ARG, "null output pointer");
  std::lock_guard<std::mutex> lock(g_mu);
  Member* M = get_member(member);
  if (!M) return fail(PDF_ERR_MEMBER, "unknown member %d", member);
  if (n == 0) return PDF_OK;
  hipError_t e = launch_locate(M->dev, x, q2, n, k, ix, iq, region, g_ncu, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch locate");
  return PDF_OK;
}

extern "C" int pdf_error_count(int64_t* count_out, int32_t reset, pdf_stream_t stream) {
  if (!count_out) return fail(PDF_ERR_ARG, "null count_out");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  unsigned long long v = 0;
  e = hipMemcpy(&v, g_nerr, sizeof v, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e, "hipMemcpy(error counter)");
  *count_out = (int64_t)v;
  if (reset) {
    e = hipMemset(g_nerr, 0, sizeof v);
    if (e != hipSuccess) return fail_hip(e, "hipMemset(error counter)");
  }
  return PDF_OK;
}

extern "C" int pdf_set_tuning(int32_t knob, int32_t value) {
  std::lock_guard<std::mutex> lock(g_mu);
  switch (knob) {
    case PDF_TUNE_LDS_POLICY:
      if (value < 0 || value > 2) return fail(PDF_ERR_ARG, "LDS policy must be 0, 1 or 2");
      g_lds_policy = value;
      return PDF_OK;
    case PDF_TUNE_VECTOR_COLUMNS:
      if (value < 0 || value > 1) return fail(PDF_ERR_ARG, "vector-columns knob must be 0 or 1");
      g_vector_cols = value;
      return PDF_OK;
    case PDF_TUNE_BLOCKS_PER_CU:
      if (value < 1 || value > 4096) return fail(PDF_ERR_ARG, "blocks per CU must be in [1, 4096]");
      g_blocks_per_cu = value;
      return PDF_OK;
    default:
      return fail(PDF_ERR_ARG, "unknown tuning knob %d", knob);
  }
}

extern "C" int pdf_get_tuning(int32_t knob, int32_t* value) {
  if (!value) return fail(PDF_ERR_ARG, "null value");
  std::lock_guard<std::mutex> lock(g_mu);
  switch (knob) {
    case PDF_TUNE_LDS_POLICY: *value = g_lds_policy; return PDF_OK;
    case PDF_TUNE_VECTOR_COLUMNS: *value = g_vector_cols; return PDF_OK;
    case PDF_TUNE_BLOCKS_PER_CU: *value = g_blocks_per_cu; return PDF_OK;
    default: return fail(PDF_ERR_ARG, "unknown tuning knob %d", knob);
  }
}

// ---------------------------------------------------------------------------------------
// Batched plans

namespace {

// The counters of the batched runs in flight (RunSlot).  A run that is queued
// takes a free one; its kernel clears the counter and writes the run's number
// to the slot's word in host memory when it has ended.  A recorded run's slot
// is its plan's until the plan is destroyed.
constexpr int kRunSlots = 4096;
constexpr int kRecordedSlots = 1024;  // at most so many of them for recorded runs
struct RunPool {
  RunSlot* dev = nullptr;      // [kRunSlots]
  unsigned* host = nullptr;    // [kRunSlots] last run that has ended in the slot (pinned)
  unsigned* done = nullptr;    // device address of host
  std::vector<unsigned> run;   // [kRunSlots] run that the slot was given to last
  std::vector<bool> kept;      // [kRunSlots] kept by a plan
  unsigned runs = 0;           // runs so far
  int next = 0, recorded = 0;
} g_runs;

// Without the pool (no memory) every run goes without a counter.
void runs_init() {
  if (g_runs.dev) return;
  RunPool p;
  hipError_t e = hipMalloc(&p.dev, sizeof(RunSlot) * kRunSlots);
  if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&p.host), sizeof(unsigned) * kRunSlots,
                                          hipHostMallocMapped | hipHostMallocCoherent);
  if (e == hipSuccess) e = hipHostGetDevicePointer(reinterpret_cast<void**>(&p.done), p.host, 0);
  if (e == hipSuccess) e = hipMemset(p.dev, 0, sizeof(RunSlot) * kRunSlots);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    if (p.dev) (void)hipFree(p.dev);
    if (p.host) (void)hipHostFree(p.host);
    (void)hipGetLastError();
    return;
  }
  std::memset(p.host, 0, sizeof(unsigned) * kRunSlots);
  p.run.assign(kRunSlots, 0);
  p.kept.assign(kRunSlots, false);
  g_runs = std::move(p);
}

bool run_ended(int slot) { return __atomic_load_n(&g_runs.host[slot], __ATOMIC_ACQUIRE) == g_runs.run[slot]; }

// Gives the slot to a new run, whose number it returns.
unsigned run_begin(int slot) {
  if (++g_runs.runs == 0) ++g_runs.runs;
  return g_runs.run[slot] = g_runs.runs;
}

// The run was not queued after all.
void run_cancel(int slot) { __atomic_store_n(&g_runs.host[slot], g_runs.run[slot], __ATOMIC_RELEASE); }

// A free slot, or -1 if none of the next few is: they are given out in turn,
// so only runs far behind, or very many, are in the way.
int run_slot() {
  for (int i = 0; g_runs.dev && i < 64; ++i) {
    const int k = g_runs.next;
    g_runs.next = (k + 1) % kRunSlots;
    if (!g_runs.kept[k] && run_ended(k)) return k;
  }
  return -1;
}

struct Plan {
  bool used = false;
  int out_f64 = 0;
  int tile_points = 4096;
  int block = 1024;  // threads of a workgroup
  int lds_block = 1024;  // the same with grids in LDS
  int vector_cols = 1;
  int use_graph = 0;
  bool lds = false;
  int max_tbl = 0;   // bytes of the largest member's location tables
  int64_t max_elems = 0;
  std::vector<BatchReq> reqs;
  std::vector<int> cols;
  std::vector<MemberDev> members;
  std::vector<std::pair<int32_t, uint64_t>> member_ids;  // (member id, load generation) behind members
  std::vector<double> invL01;
  int ntiles = 0;
  void* dmem = nullptr;        // reqs, cols, members, invL01
  BatchTile* d_tiles = nullptr;
  int tiles_cap = 0;
  BatchReq* d_reqs = nullptr;
  int* d_cols = nullptr;
  MemberDev* d_members = nullptr;
  double* d_invL01 = nullptr;
  std::vector<int> kept;           // slots of recorded runs
  void* compact = nullptr;         // compacted copies of members' values (FP64 plans)
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  int exec_slot = -1;
  // kernel argument storage (addresses handed to hipLaunchKernel / graph nodes)
  RunSlot* a_slot = nullptr;
  unsigned* a_done = nullptr;
  unsigned a_run = 0;
  int a_ntiles = 0, a_max_tbl = 0, a_vec = 0;
  void* args[12];
};

std::vector<Plan> g_plans;

void plan_free_graph(Plan& P) {
  if (P.exec) (void)hipGraphExecDestroy(P.exec);
  if (P.graph) (void)hipGraphDestroy(P.graph);
  P.exec = nullptr;
  P.graph = nullptr;
}

void plan_release(Plan& P) {
  plan_free_graph(P);
  if (P.dmem) (void)hipFree(P.dmem);  // waits for the device: no run of the plan is in flight after it
  if (P.d_tiles) (void)hipFree(P.d_tiles);
  if (P.compact) (void)hipFree(P.compact);
  for (int k : P.kept) {
    g_runs.kept[k] = false;
    run_cancel(k);
    --g_runs.recorded;
  }
  P = Plan();
}

// (Re)build the tile list for the plan's tile size and upload it.  The device
// is drained first: a run of this plan still in flight on some stream reads
// the tile list being replaced.
int plan_tiles(Plan& P) {
  if (P.d_tiles) {
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return fail_hip(e, "hipDeviceSynchronize");
  }
  std::vector<BatchTile> t;
  // tiles grouped by member so that consecutive tiles tend to share a staged grid
  std::vector<int> order(P.reqs.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return P.reqs[a].member < P.reqs[b].member; });
  std::vector<TileReq> sizes;
  for (const BatchReq& r : P.reqs) sizes.push_back(TileReq{r.n, r.R});
  const BatchTiling cut = batch_tiling(P.lds, P.tile_points, sizes, g_ncu);
  P.block = P.lds ? P.lds_block : cut.block;
  for (int r : order) {
    const int64_t n = P.reqs[r].n;
    // workgroups of one tile each: a request's tiles alike (700 points as 384
    // and 316, not 512 and 188); else the remainders fill the end of the run
    const int64_t k = (n + cut.points - 1) / cut.points;
    const int64_t tp = P.block != kBatchHalf || k == 0 ? cut.points : ((n + k - 1) / k + 63) / 64 * 64;
    for (int64_t s0 = 0; s0 < n; s0 += tp) t.push_back(BatchTile{r, (int)std::min<int64_t>(tp, n - s0), s0});
  }
  if ((int64_t)t.size() > (1LL << 30)) return fail(PDF_ERR_ARG, "too many tiles");
  // one tile per workgroup: dealt out by cost, points times columns (46 requests
  // of 1000 to 15900 points and 1 to 11 columns, FP64: 22.8 us in request order,
  // 20.4 so, 20.8 one by one; 50 requests of 5000 points and 13 columns, 50
  // members: 34, 34 and 69 us)
  if (P.block == kBatchHalf) {
    std::vector<int64_t> cost;
    for (const BatchTile& b : t) cost.push_back((int64_t)b.count * P.reqs[b.req].R);
    std::vector<BatchTile> dealt;
    for (size_t i : deal_tiles(cost)) dealt.push_back(t[i]);
    t.swap(dealt);
  }
  // the costliest tiles first (points times groups of four columns), so that
  // the workgroups end together on small ones; equal tiles stay grouped.  Not
  // where the grids are read from global memory: there a request's tiles belong
  // together, as they find its member's rows in the caches (100 requests of
  // 30000 points, 13 columns, FP64: 554 us costliest first, 495 in order)
  if (P.lds)
    std::stable_sort(t.begin(), t.end(), [&](const BatchTile& a, const BatchTile& b) {
      return (int64_t)a.count * ((P.reqs[a.req].R + 3) / 4) > (int64_t)b.count * ((P.reqs[b.req].R + 3) / 4);
    });
  P.ntiles = (int)t.size();
  if (P.ntiles > P.tiles_cap) {
    if (P.d_tiles) (void)hipFree(P.d_tiles);
    P.d_tiles = nullptr;
    hipError_t e = hipMalloc(&P.d_tiles, sizeof(BatchTile) * std::max(1, P.ntiles));
    if (e != hipSuccess) return fail_hip(e, "hipMalloc(tiles)");
    P.tiles_cap = P.ntiles;
  }
  if (P.ntiles) {
    hipError_t e = hipMemcpy(P.d_tiles, t.data(), sizeof(BatchTile) * t.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail_hip(e, "hipMemcpy(tiles)");
  }
  return PDF_OK;
}

BatchLaunch plan_params(const Plan& P) {
  return batch_launch_params(!P.out_f64, P.lds, P.max_tbl, P.max_elems, g_ncu, P.ntiles, P.block);
}

// Kernel arguments of a run with counter `slot` (-1: none).
void plan_args(Plan& P, int slot) {
  P.a_slot = slot < 0 ? nullptr : g_runs.dev + slot;
  P.a_done = slot < 0 ? nullptr : g_runs.done + slot;
  P.a_run = slot < 0 ? 0 : run_begin(slot);
  P.a_ntiles = P.ntiles;
  P.a_max_tbl = P.max_tbl;
  P.a_vec = P.vector_cols;
  P.args[0] = &P.d_reqs;
  P.args[1] = &P.d_cols;
  P.args[2] = &P.d_tiles;
  P.args[3] = &P.a_ntiles;
  P.args[4] = &P.d_members;
  P.args[5] = &P.d_invL01;
  P.args[6] = &P.a_slot;
  P.args[7] = &P.a_done;
  P.args[8] = &P.a_run;
  P.args[9] = &g_nerr;
  P.args[10] = &P.a_max_tbl;
  P.args[11] = &P.a_vec;
}

// A slot that the plan keeps for a recorded run, or -1.
int plan_keep_slot(Plan& P) {
  const int k = g_runs.recorded < kRecordedSlots ? run_slot() : -1;
  if (k < 0) return -1;
  P.kept.push_back(k);
  g_runs.kept[k] = true;
  ++g_runs.recorded;
  return k;
}

int plan_build_graph(Plan& P, const BatchLaunch& L) {
  plan_free_graph(P);
  hipError_t e = batch_prepare(L);
  if (e != hipSuccess) return fail_hip(e, "hipFuncSetAttribute(batched)");
  if (P.exec_slot >= 0 && !run_ended(P.exec_slot)) P.exec_slot = -1;  // a run of an earlier graph still has it
  if (L.counted && P.exec_slot < 0) P.exec_slot = plan_keep_slot(P);
  plan_args(P, L.counted ? P.exec_slot : -1);
  if (L.counted && P.exec_slot >= 0) run_cancel(P.exec_slot);  // recorded, not in flight
  if ((e = hipGraphCreate(&P.graph, 0)) != hipSuccess) return fail_hip(e, "hipGraphCreate");
  hipKernelNodeParams k{};
  k.func = const_cast<void*>(L.main_fn);
  k.gridDim = dim3(L.grid);
  k.blockDim = dim3(L.block);
  k.sharedMemBytes = (unsigned)L.shm;
  k.kernelParams = P.args;
  hipGraphNode_t node;
  if ((e = hipGraphAddKernelNode(&node, P.graph, nullptr, 0, &k)) != hipSuccess) return fail_hip(e, "graph node");
  if ((e = hipGraphInstantiate(&P.exec, P.graph, nullptr, nullptr, 0)) != hipSuccess)
    return fail_hip(e, "hipGraphInstantiate");
  return PDF_OK;
}

int plan_run(Plan& P, hipStream_t s) {
  if (P.ntiles == 0) return PDF_OK;
  const BatchLaunch L = plan_params(P);
  const bool recording = L.counted && capturing(s);
  // the plan's graph holds one counter: a run that finds it in flight is queued plainly
  if (P.use_graph && !recording) {
    if (!P.exec) {
      const int rc = plan_build_graph(P, L);
      if (rc != PDF_OK) return rc;
    }
    const int k = L.counted ? P.exec_slot : -1;
    if (k < 0 || run_ended(k)) {
      if (k >= 0) __atomic_store_n(&g_runs.host[k], 0u, __ATOMIC_RELEASE);
      const hipError_t e = hipGraphLaunch(P.exec, s);
      if (e == hipSuccess) return PDF_OK;
      if (k >= 0) run_cancel(k);
      return fail_hip(e, "hipGraphLaunch");
    }
  }
  const int k = !L.counted ? -1 : recording ? plan_keep_slot(P) : run_slot();
  plan_args(P, k);
  hipError_t e = batch_prepare(L);
  if (e == hipSuccess) e = batch_launch(L, P.args, s);
  if (e == hipSuccess) return PDF_OK;
  if (k >= 0) run_cancel(k);
  return fail_hip(e, "launch batched");
}

Plan* get_plan(int32_t id) {
  if (id < 0 || id >= (int32_t)g_plans.size() || !g_plans[id].used) return nullptr;
  return &g_plans[id];
}

// A plan holds copies of its members' device pointers: every member must still
// be the one loaded when the plan was built (not unloaded, slot not reused).
int plan_members_live(const Plan& P) {
  for (const auto& mg : P.member_ids) {
    const Member* M = get_member(mg.first);
    if (!M || M->gen != mg.second)
      return fail(PDF_ERR_MEMBER, "member %d was unloaded after the plan was built", mg.first);
  }
  return PDF_OK;
}

// Autotune choices (tile points, vector columns) by request signature and
// device, and the file they are also kept in ("" = none).
std::map<std::string, std::pair<int, int>> g_tune_cache;
std::string g_tune_path;

bool valid_tile(int tile) { return tile >= 64 && tile <= (1 << 22) && (tile & 63) == 0; }

// Reads the "key tile vector" lines of a cache file into g_tune_cache; lines
// that do not parse or hold an invalid choice are skipped.  A missing file
// holds no entries.
int tune_cache_load(const char* path) {
  FILE* f = std::fopen(path, "r");
  if (!f) return errno == ENOENT ? PDF_OK : fail(PDF_ERR_ARG, "cannot read autotune cache %s", path);
  char line[512], key[400];
  while (std::fgets(line, sizeof line, f)) {
    int tile = 0, vec = -1;
    if (std::sscanf(line, "%399s %d %d", key, &tile, &vec) == 3 && valid_tile(tile) && (vec == 0 || vec == 1))
      g_tune_cache[key] = {tile, vec};
  }
  std::fclose(f);
  return PDF_OK;
}

}  // namespace

extern "C" int pdf_batch_tune_cache(const char* path) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (!path || !*path) {
    g_tune_path.clear();
    return PDF_OK;
  }
  const int rc = tune_cache_load(path);
  if (rc != PDF_OK) return rc;
  g_tune_path = path;
  return PDF_OK;
}

namespace {
// Plans with FP64 outputs read the grids from global memory: a request for
// some of the stored flavours, or in another order, or with absent ones, gets
// a copy of the member's values compacted to it (see Layout), so that it is
// walked in 16-byte groups.  The plan keeps the copies, at most kPlanCompact
// bytes; requests beyond that, and one-shot calls, read the member's rows.
constexpr size_t kPlanCompact = (size_t)256 << 20;

struct PlanBuilder {
  std::map<int, int> slot;  // member id -> plan member index
  std::map<std::pair<int, std::vector<int>>, int> layouts;  // (plan member, column list) -> layout number
  std::map<std::pair<int, std::vector<int>>, int> copies;   // the same -> plan member index of the compacted copy
  size_t copied = 0;
  int64_t compact_elems = 0;

  int add_member(Plan& P, const MemberDev& d, const Member& M) {
    P.members.push_back(d);
    P.invL01.push_back(M.invL01);
    P.max_tbl = std::max(P.max_tbl, d.tbl_bytes);
    P.max_elems = std::max(P.max_elems, P.out_f64 ? d.elems64 : d.elems32);
    return (int)P.members.size() - 1;
  }

  std::vector<CompactJob> jobs;
  std::vector<int> job_member;  // plan member index of each job's copy

  // Plan member index of the copy for this request, or -1 to read the member's
  // rows.  Rows of an even number of values (16-byte groups stay aligned where
  // the grids fit LDS), never longer than the member's own.
  int copy_of(Plan& P, int member, const Member& M, const ReqCols& rc, const std::vector<int>& list) {
    const auto key = std::make_pair(member, list);
    const auto it = copies.find(key);
    if (it != copies.end()) return it->second;
    const int stride = rc.n > 12 ? (rc.n + 15) & ~15 : (rc.n + 1) & ~1;
    const size_t bytes = align_up((size_t)M.dev.rows * stride * sizeof(double), 256);
    if (stride > M.dev.P64 || copied + bytes > kPlanCompact) return -1;
    MemberDev d = M.dev;
    d.P = rc.n;
    d.P64 = stride;
    d.elems64 = (int64_t)M.dev.rows * stride;
    const int to = add_member(P, d, M);
    jobs.push_back({M.dev.v64, nullptr, d.elems64, M.dev.P64, stride, rc});
    job_member.push_back(to);
    copied += bytes;
    return copies[key] = to;
  }

  // Allocates the copies; the jobs fill them.
  hipError_t allocate(Plan& P) {
    if (jobs.empty()) return hipSuccess;
    const hipError_t e = hipMalloc(&P.compact, copied);
    if (e != hipSuccess) return e;
    unsigned char* at = static_cast<unsigned char*>(P.compact);
    for (size_t i = 0; i < jobs.size(); ++i) {
      jobs[i].dst = reinterpret_cast<double*>(at);
      P.members[job_member[i]].v64 = jobs[i].dst;
      at += align_up((size_t)jobs[i].elems * sizeof(double), 256);
    }
    return hipSuccess;
  }
};

constexpr int kRetryPlain = 1;  // no memory for the copies: build the plan without them

int batch_create(const pdf_request* reqs, int32_t n_req, int32_t out_f64, bool copies, int32_t* plan_out) {
  if (!plan_out || (n_req > 0 && !reqs) || n_req < 0) return fail(PDF_ERR_ARG, "bad argument");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  runs_init();
  Plan P;
  P.used = true;
  P.out_f64 = out_f64 ? 1 : 0;
  PlanBuilder B;
  for (int i = 0; i < n_req; ++i) {
    const pdf_request& q = reqs[i];
    Member* M = get_member(q.member);
    if (q.n < 0)
      rc = fail(PDF_ERR_ARG, "request %d: n < 0", i);
    else if (q.n > 0 && (!q.x || !q.q2 || !q.out))
      rc = fail(PDF_ERR_ARG, "request %d: null device pointer", i);
    else if (!M)
      rc = fail(PDF_ERR_MEMBER, "request %d: unknown member %d", i, q.member);
    if (rc != PDF_OK) return rc;
    ReqCols rcols{};
    if ((rc = build_req(*M, q.pids, q.n_pids, rcols)) != PDF_OK) return rc;
    if (!B.slot.count(q.member)) {
      B.slot[q.member] = B.add_member(P, M->dev, *M);
      P.member_ids.push_back({q.member, M->gen});
    }
    BatchReq b{};
    b.member = B.slot[q.member];
    b.R = rcols.n;
    b.col_off = (int)P.cols.size();
    b.all_cols = rcols.n == M->dev.P;
    std::vector<int> list(rcols.col, rcols.col + rcols.n), pos((size_t)M->dev.P, -1);
    bool compact = !P.out_f64 && rcols.n <= kCompactCols;
    for (int j = 0; j < rcols.n; ++j) {
      if (list[j] != j) b.all_cols = 0;
      if (list[j] < 0) continue;
      if (pos[list[j]] >= 0) compact = false;  // a flavour requested twice has two output positions
      pos[list[j]] = j;
    }
    P.cols.insert(P.cols.end(), list.begin(), list.end());
    b.layout = -1;
    if (compact) {
      P.cols.insert(P.cols.end(), pos.begin(), pos.end());
      b.layout = B.layouts.insert({{b.member, list}, (int)B.layouts.size()}).first->second;
      B.compact_elems = std::max(B.compact_elems, (int64_t)M->dev.rows * kCompactCols);
    }
    if (copies && g_vector_cols && P.out_f64 && !b.all_cols && b.R >= 2 && q.n > 0) {
      const int c = B.copy_of(P, b.member, *M, rcols, list);
      if (c >= 0) {
        b.member = c;
        b.all_cols = 1;
        for (int j = 0; j < b.R; ++j)
          if (list[j] >= 0) P.cols[b.col_off + j] = j;
      }
    }
    b.x = q.x;
    b.q2 = q.q2;
    b.out = q.out;
    b.n = q.n;
    P.reqs.push_back(b);
  }
  if (B.allocate(P) != hipSuccess) {
    (void)hipGetLastError();
    plan_release(P);
    return kRetryPlain;
  }
  // the grids in LDS where the largest fits beside the records of 16 waves, or
  // of 12 if there is more than a round of half-size workgroups to do (30
  // requests of 3000 points on 100 x 51 x 2 values in FP32, all outside the grid:
  // 21 us, from global memory 15; of 100000 points inside it: 70 and 156)
  int64_t half = 0;
  for (const BatchReq& r : P.reqs) half += (r.n + 511) / 512;
  auto fits = [&](int64_t elems, int block) {
    return batch_shared_bytes(P.max_tbl, !P.out_f64, true, block) + (size_t)elems * (P.out_f64 ? 8 : 4) <= kLdsBytes - 1024;
  };
  P.lds_block = fits(P.max_elems, kBatchThreads) ? kBatchThreads : kBatchSmall;
  P.lds = g_lds_policy != 1 && fits(P.max_elems, P.lds_block) &&
          (P.lds_block == kBatchThreads || g_lds_policy == 2 || half > 2 * (int64_t)g_ncu);
  // compacted layouts when their rows fit LDS too
  if (P.lds && B.compact_elems > P.max_elems) {
    if (fits(B.compact_elems, P.lds_block))
      P.max_elems = B.compact_elems;
    else
      for (BatchReq& b : P.reqs) b.layout = -1;
  }
  // requests, columns, members, jobs of the copies: one block, one transfer
  size_t bytes = 0;
  auto part = [&](size_t n) {
    const size_t at = bytes;
    bytes += align_up(std::max<size_t>(1, n), 256);
    return at;
  };
  const size_t br = part(sizeof(BatchReq) * P.reqs.size()), bc = part(sizeof(int) * P.cols.size());
  const size_t bm = part(sizeof(MemberDev) * P.members.size()), bi = part(sizeof(double) * P.invL01.size());
  const size_t bj = part(sizeof(CompactJob) * B.jobs.size());
  std::vector<unsigned char> blob(bytes);
  auto put = [&](size_t at, const auto& v) {
    if (!v.empty()) std::memcpy(blob.data() + at, v.data(), sizeof(v[0]) * v.size());
  };
  put(br, P.reqs);
  put(bc, P.cols);
  put(bm, P.members);
  put(bi, P.invL01);
  put(bj, B.jobs);
  hipError_t e = hipMalloc(&P.dmem, bytes);
  if (e == hipSuccess) e = hipMemcpy(P.dmem, blob.data(), bytes, hipMemcpyHostToDevice);
  unsigned char* b = static_cast<unsigned char*>(P.dmem);
  if (e == hipSuccess && !B.jobs.empty()) {
    int64_t most = 0;
    for (const CompactJob& j : B.jobs) most = std::max(most, j.elems);
    e = launch_compact_jobs(reinterpret_cast<const CompactJob*>(b + bj), (int)B.jobs.size(), most, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  }
  if (e != hipSuccess) {
    plan_release(P);
    return fail_hip(e, "plan tables");
  }
  P.d_reqs = reinterpret_cast<BatchReq*>(b + br);
  P.d_cols = reinterpret_cast<int*>(b + bc);
  P.d_members = reinterpret_cast<MemberDev*>(b + bm);
  P.d_invL01 = reinterpret_cast<double*>(b + bi);
  if ((rc = plan_tiles(P)) != PDF_OK) {
    plan_release(P);
    return rc;
  }
  for (size_t i = 0; i < g_plans.size(); ++i)
    if (!g_plans[i].used) {
      g_plans[i] = P;
      *plan_out = (int32_t)i;
      return PDF_OK;
    }
  g_plans.push_back(P);
  *plan_out = (int32_t)(g_plans.size() - 1);
  return PDF_OK;
}

}  // namespace

extern "C" int pdf_batch_create(const pdf_request* reqs, int32_t n_req, int32_t out_f64, int32_t* plan_out) {
  const int rc = batch_create(reqs, n_req, out_f64, true, plan_out);  // with copies unless declined
  return rc == kRetryPlain ? batch_create(reqs, n_req, out_f64, false, plan_out) : rc;
}

extern "C" int pdf_batch_configure(int32_t plan, int32_t tile_points, int32_t vector_cols, int32_t use_graph) {
  std::lock_guard<std::mutex> lock(g_mu);
  Plan* P = get_plan(plan);
  if (!P) return fail(PDF_ERR_ARG, "unknown plan %d", plan);
  if (tile_points < 64 || tile_points > (1 << 22) || (tile_points & 63))
    return fail(PDF_ERR_ARG, "tile_points must be a multiple of 64 in [64, 4194304]");
  if (vector_cols < 0 || vector_cols > 1 || use_graph < 0 || use_graph > 1)
    return fail(PDF_ERR_ARG, "flags must be 0 or 1");
  plan_free_graph(*P);
  P->vector_cols = vector_cols;
  P->use_graph = use_graph;
  if (tile_points != P->tile_points) {
    P->tile_points = tile_points;
    return plan_tiles(*P);
  }
  return PDF_OK;
}

extern "C" int pdf_batch_run(int32_t plan, pdf_stream_t stream) {
  std::lock_guard<std::mutex> lock(g_mu);
  Plan* P = get_plan(plan);
  if (!P) return fail(PDF_ERR_ARG, "unknown plan %d", plan);
  const int rc = plan_members_live(*P);
  if (rc != PDF_OK) return rc;
  return plan_run(*P, (hipStream_t)stream);
}

extern "C" int pdf_batch_autotune(int32_t plan, int32_t reps, pdf_stream_t stream, int32_t* tile_out,
                                  int32_t* vector_out) {
  if (reps < 1) return fail(PDF_ERR_ARG, "reps must be >= 1");
  std::lock_guard<std::mutex> lock(g_mu);
  Plan* P = get_plan(plan);
  if (!P) return fail(PDF_ERR_ARG, "unknown plan %d", plan);
  if (plan_members_live(*P) != PDF_OK) return PDF_ERR_MEMBER;
  hipStream_t s = (hipStream_t)stream;
  // signature of the work: request count, point total, flavour total, precision
  int64_t pts = 0, evals = 0;
  for (auto& r : P->reqs) {
    pts += r.n;
    evals += r.n * r.R;
  }
  char key[400];
  snprintf(key, sizeof key, "%s/%d/%zu/%lld/%lld/%d/%d", g_arch.c_str(), g_ncu, P->reqs.size(), (long long)pts,
           (long long)evals, P->out_f64, (int)P->lds);
  auto it = g_tune_cache.find(key);
  int best_tile = P->tile_points, best_vec = P->vector_cols;
  if (it != g_tune_cache.end()) {
    best_tile = it->second.first;
    best_vec = it->second.second;
  } else {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const int saved_graph = P->use_graph;
    // the sweep; every exit path below restores the plan's graph flag and frees the events
    auto sweep = [&]() -> int {
      if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return fail(PDF_ERR_DEVICE, "hipEventCreate");
      float best = 1e30f;
      P->use_graph = 0;
      for (int tp : {1024, 2048, 4096, 8192, 16384}) {
        for (int vec : {0, 1}) {
          P->tile_points = tp;
          P->vector_cols = vec;
          int rc = plan_tiles(*P);
          if (rc != PDF_OK) return rc;
          if ((rc = plan_run(*P, s)) != PDF_OK) return rc;  // warm-up
          float tot = 0.0f;
          for (int r = 0; r < reps; ++r) {
            (void)hipEventRecord(e0, s);
            if ((rc = plan_run(*P, s)) != PDF_OK) return rc;
            (void)hipEventRecord(e1, s);
            if (hipEventSynchronize(e1) != hipSuccess) return fail(PDF_ERR_DEVICE, "hipEventSynchronize");
            float ms = 0.0f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            tot += ms;
          }
          if (tot < best) {
            best = tot;
            best_tile = tp;
            best_vec = vec;
          }
        }
      }
      return PDF_OK;
    };
    const int rc = sweep();
    P->use_graph = saved_graph;
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (rc != PDF_OK) return rc;
    g_tune_cache[key] = {best_tile, best_vec};
    if (!g_tune_path.empty()) {  // best effort: a cache that cannot be written only costs a later sweep
      if (FILE* f = std::fopen(g_tune_path.c_str(), "a")) {
        std::fprintf(f, "%s %d %d\n", key, best_tile, best_vec);
        std::fclose(f);
      }
    }
  }
  plan_free_graph(*P);
  P->tile_points = best_tile;
  P->vector_cols = best_vec;
  int rc = plan_tiles(*P);
  if (rc != PDF_OK) return rc;
  if (tile_out) *tile_out = best_tile;
  if (vector_out) *vector_out = best_vec;
  return PDF_OK;
}

extern "C" int pdf_batch_destroy(int32_t plan) {
  std::lock_guard<std::mutex> lock(g_mu);
  Plan* P = get_plan(plan);
  if (!P) return fail(PDF_ERR_ARG, "unknown plan %d", plan);
  plan_release(*P);
  return PDF_OK;
}

namespace {
int batched_one_shot(const pdf_request* reqs, int32_t n_req, int32_t out_f64, pdf_stream_t stream) {
  int32_t plan = -1;
  int rc = batch_create(reqs, n_req, out_f64, false, &plan);
  if (rc != PDF_OK) return rc;
  rc = pdf_batch_run(plan, stream);
  if (rc == PDF_OK) {
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) rc = fail_hip(e, "hipStreamSynchronize");
  }
  pdf_batch_destroy(plan);
  return rc;
}
}  // namespace

extern "C" int pdf_xfxq2_batched(const pdf_request* reqs, int32_t n_req, pdf_stream_t stream) {
  return batched_one_shot(reqs, n_req, 0, stream);
}

extern "C" int pdf_xfxq2_batched_f64(const pdf_request* reqs, int32_t n_req, pdf_stream_t stream) {
  return batched_one_shot(reqs, n_req, 1, stream);
}

// ---------------------------------------------------------------------------------------
// MLP surrogates

namespace {

struct Surrogate {
  bool used = false;
  int member = -1;
  uint64_t member_gen = 0;   // load generation of the member the surrogate was built on
  SurDev sd{};
  SurBufs b{};
  void* pmem = nullptr;      // parameters, moments, gradients, envelope tables
  void* bmem = nullptr;      // training workspace (sized for batches of up to bcap rows)
  int bcap = 0;
  float* d_in = nullptr;     // training inputs [n][2]
  float* d_t = nullptr;      // training targets [n][kO]
  int64_t n_train = 0;
  int64_t step = 0;          // Adam steps taken
  uint64_t seed = 0;
  // training steps recorded as graphs, valid for g_batch and g_in: kGraphSteps steps, and one step for what is left
  hipStream_t cap = nullptr;
  hipGraph_t graph[2] = {};
  hipGraphExec_t exec[2] = {};
  int g_batch = 0;
  const float* g_in = nullptr;
  const void* g_bmem = nullptr;
};

// Steps per replay of the long training graph: between the kernels of one
// replay the GPU waits about 1 us, between two replays the host's launch cost
// shows (batch 4096, per step: 18.9 us with one step per replay, 14.5 us with 16).
constexpr int kGraphSteps[2] = {16, 1};

std::vector<Surrogate> g_surs;

Surrogate* get_sur(int32_t id) {
  if (id < 0 || id >= (int32_t)g_surs.size() || !g_surs[id].used) return nullptr;
  return &g_surs[id];
}

// The surrogate's member, or null once it was unloaded (or its slot reused).
Member* sur_member(const Surrogate& S) {
  Member* M = get_member(S.member);
  return M && M->gen == S.member_gen ? M : nullptr;
}

void sur_free_graph(Surrogate& S) {
  for (int k = 0; k < 2; ++k) {
    if (S.exec[k]) (void)hipGraphExecDestroy(S.exec[k]);
    if (S.graph[k]) (void)hipGraphDestroy(S.graph[k]);
    S.exec[k] = nullptr;
    S.graph[k] = nullptr;
  }
  S.g_batch = 0;
  S.g_in = nullptr;
  S.g_bmem = nullptr;
}

void sur_release(Surrogate& S) {
  sur_free_graph(S);
  if (S.cap) (void)hipStreamDestroy(S.cap);
  if (S.pmem) (void)hipFree(S.pmem);
  if (S.bmem) (void)hipFree(S.bmem);
  if (S.d_in) (void)hipFree(S.d_in);
  S = Surrogate();
}

uint64_t splitmix64(uint64_t& x) {
  uint64_t z = (x += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Glorot-uniform weights, zero biases, from a counter-based generator.
std::vector<float> sur_init_params(uint64_t seed) {
  const int H = sur_hidden(), O = sur_out_width();
  std::vector<float> p((size_t)sur_nparams(), 0.0f);
  uint64_t st = seed;
  auto fill = [&](size_t off, int fan_out, int fan_in) {
    const double a = std::sqrt(6.0 / (fan_in + fan_out));
    for (int i = 0; i < fan_out * fan_in; ++i) {
      const double u = (double)(splitmix64(st) >> 11) * (1.0 / 9007199254740992.0);
      p[off + i] = (float)((2.0 * u - 1.0) * a);
    }
  };
  size_t off = 0;
  fill(off, H, 2); off += (size_t)H * 2 + H;
  fill(off, H, H); off += (size_t)H * H + H;
  fill(off, H, H); off += (size_t)H * H + H;
  fill(off, O, H);
  return p;
}

int sur_ensure_batch(Surrogate& S, int B) {
  if (B <= S.bcap) return PDF_OK;
  if (S.bmem) (void)hipFree(S.bmem);
  S.bmem = nullptr;
  // the fused training step's per-slice partial gradients and losses
  hipError_t e = hipMalloc(&S.bmem, sur_workspace_floats(B) * 4);
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(surrogate batch)");
  S.b.wpart = static_cast<float*>(S.bmem);
  S.bcap = B;
  return PDF_OK;
}

// Records graph k: kGraphSteps[k] training steps on batches of `batch` rows.
int sur_record_steps(Surrogate& S, int batch, int k) {
  hipError_t e = hipSuccess;
  if (!S.cap && (e = hipStreamCreateWithFlags(&S.cap, hipStreamNonBlocking)) != hipSuccess)
    return fail_hip(e, "hipStreamCreate(capture)");
  if ((e = hipStreamBeginCapture(S.cap, hipStreamCaptureModeThreadLocal)) != hipSuccess)
    return fail_hip(e, "hipStreamBeginCapture");
  hipError_t e1 = hipSuccess;
  for (int i = 0; i < kGraphSteps[k] && e1 == hipSuccess; ++i) e1 = sur_train_step(S.b, S.d_in, S.d_t, batch, S.cap);
  e = hipStreamEndCapture(S.cap, &S.graph[k]);
  if (e1 != hipSuccess || e != hipSuccess) {
    sur_free_graph(S);
    return fail_hip(e1 != hipSuccess ? e1 : e, "capture of a training step");
  }
  if ((e = hipGraphInstantiate(&S.exec[k], S.graph[k], nullptr, nullptr, 0)) != hipSuccess) {
    sur_free_graph(S);
    return fail_hip(e, "hipGraphInstantiate(training step)");
  }
  S.g_batch = batch;
  S.g_in = S.d_in;
  S.g_bmem = S.bmem;
  return PDF_OK;
}

constexpr char kSurMagic[8] = {'P', 'D', 'F', 'M', 'I', 'S', 'R', '1'};

uint64_t fnv1a(const unsigned char* p, size_t n, uint64_t h = 1469598103934665603ull) {
  for (size_t i = 0; i < n; ++i) {
    h ^= p[i];
    h *= 1099511628211ull;
  }
  return h;
}

}  // namespace

extern "C" int pdf_surrogate_param_count(int32_t* n_out) {
  if (!n_out) return fail(PDF_ERR_ARG, "null n_out");
  *n_out = sur_nparams();
  return PDF_OK;
}

extern "C" int pdf_surrogate_create(int32_t member, uint64_t seed, int32_t* sid_out) {
  if (!sid_out) return fail(PDF_ERR_ARG, "null sid_out");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  Member* M = get_member(member);
  if (!M) return fail(PDF_ERR_MEMBER, "unknown member %d", member);
  const int O = sur_out_width(), NP = sur_nparams();
  const int P = (int)M->pids.size();
  if (P > O) return fail(PDF_ERR_ARG, "surrogate supports at most %d stored flavours", O);
  const int K = (int)M->h_shape.size() / 2;
  const int nx0 = M->h_shape[0];
  const double* xk0 = M->h_knots.data();
  // envelope over sub-grid 0's x knots: at each, the value of largest magnitude over every Q^2 knot of every
  // sub-grid (signed); slopes d E / d ln x by finite differences (mean of the adjacent secants, one-sided at
  // the ends)
  std::vector<double> envv((size_t)nx0 * O, 0.0), enva((size_t)nx0 * O, -1.0), lxk(nx0);
  for (int i = 0; i < nx0; ++i) lxk[i] = std::log(xk0[i]);
  int64_t ko = 0, vo = 0;
  for (int k = 0; k < K; ++k) {
    const int nx = M->h_shape[2 * k], nq = M->h_shape[2 * k + 1];
    const double* xk = M->h_knots.data() + ko;
    for (int ix = 0; ix < nx; ++ix) {
      int i0 = 0;  // nearest sub-grid-0 knot
      for (int j = 0; j < nx0; ++j)
        if (std::fabs(std::log(xk0[j] / xk[ix])) < std::fabs(std::log(xk0[i0] / xk[ix]))) i0 = j;
      for (int iq = 0; iq < nq; ++iq)
        for (int c = 0; c < P; ++c) {
          const double v = M->h_values[vo + ((int64_t)ix * nq + iq) * P + c];
          if (std::fabs(v) > enva[(size_t)i0 * O + c]) {
            enva[(size_t)i0 * O + c] = std::fabs(v);
            envv[(size_t)i0 * O + c] = v;
          }
        }
    }
    ko += nx + nq;
    vo += (int64_t)nx * nq * P;
  }
  std::vector<float> env((size_t)nx0 * O), envd((size_t)nx0 * O);
  for (int i = 0; i < nx0; ++i)
    for (int c = 0; c < O; ++c) {
      auto sec = [&](int j) {  // secant over cell j
        return (envv[(size_t)(j + 1) * O + c] - envv[(size_t)j * O + c]) / (lxk[j + 1] - lxk[j]);
      };
      const double d = i == 0 ? sec(0) : i == nx0 - 1 ? sec(nx0 - 2) : 0.5 * (sec(i - 1) + sec(i));
      env[(size_t)i * O + c] = (float)envv[(size_t)i * O + c];
      envd[(size_t)i * O + c] = (float)d;
    }
  Surrogate S;
  S.used = true;
  S.member = member;
  S.member_gen = M->gen;
  S.seed = seed;
  S.sd.P = P;
  S.sd.nx = nx0;
  S.sd.K = K;
  S.sd.lx0 = std::log(M->dev.xmin);
  S.sd.ilx = 1.0 / (std::log(M->dev.xmax) - std::log(M->dev.xmin));
  S.sd.lq0 = std::log(M->dev.qmin);
  S.sd.ilq = 1.0 / (std::log(M->dev.qmax) - std::log(M->dev.qmin));
  if (nx0 > kSurMaxEnvKnots)
    return fail(PDF_ERR_GRID, "surrogate envelope supports at most %d x knots", kSurMaxEnvKnots);
  {
    int64_t o = 0;
    for (int k = 0; k < K; ++k) {
      const int nx = M->h_shape[2 * k], nq = M->h_shape[2 * k + 1];
      const double* xk = M->h_knots.data() + o;
      const double* qk = xk + nx;
      S.sd.qfirst[k] = qk[0];
      S.sd.trust[k] = nx >= 4 && nq >= 4;
      S.sd.txlo[k] = S.sd.trust[k] ? xk[1] : 0.0;
      S.sd.txhi[k] = S.sd.trust[k] ? xk[nx - 2] : 0.0;
      S.sd.tqlo[k] = S.sd.trust[k] ? qk[1] : 0.0;
      S.sd.tqhi[k] = S.sd.trust[k] ? qk[nq - 2] : 0.0;
      o += nx + nq;
    }
  }
  const size_t bp = align_up((size_t)NP * 4, 256), bpb = align_up((size_t)sur_halves() * 2, 256);
  const size_t be = align_up(env.size() * 4, 256), bl = align_up(lxk.size() * 8, 256);
  hipError_t e = hipMalloc(&S.pmem, 4 * bp + bpb + 2 * be + bl + 2048 + align_up(sizeof(SurStep), 256));
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(surrogate)");
  unsigned char* b = static_cast<unsigned char*>(S.pmem);
  S.b.P = reinterpret_cast<float*>(b);
  S.b.M = reinterpret_cast<float*>(b + bp);
  S.b.V = reinterpret_cast<float*>(b + 2 * bp);
  S.b.G = reinterpret_cast<float*>(b + 3 * bp);
  S.b.Pb = reinterpret_cast<unsigned short*>(b + 4 * bp);
  float* envdev = reinterpret_cast<float*>(b + 4 * bp + bpb);
  float* envddev = reinterpret_cast<float*>(b + 4 * bp + bpb + be);
  double* lxkd = reinterpret_cast<double*>(b + 4 * bp + bpb + 2 * be);
  S.b.loss = reinterpret_cast<float*>(b + 4 * bp + bpb + 2 * be + bl);
  S.b.st = reinterpret_cast<SurStep*>(b + 4 * bp + bpb + 2 * be + bl + 2048);
  S.sd.env = envdev;
  S.sd.envd = envddev;
  S.sd.lxk = lxkd;
  const std::vector<float> p0 = sur_init_params(seed);
  std::vector<float> zeros((size_t)NP, 0.0f);
  if ((e = hipMemcpy(S.b.P, p0.data(), (size_t)NP * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(S.b.M, zeros.data(), (size_t)NP * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(S.b.V, zeros.data(), (size_t)NP * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(envdev, env.data(), env.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(envddev, envd.data(), envd.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(lxkd, lxk.data(), lxk.size() * 8, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = sur_refresh_bf16(S.b, nullptr)) != hipSuccess || (e = hipDeviceSynchronize()) != hipSuccess) {
    sur_release(S);
    return fail_hip(e, "surrogate upload");
  }
  for (size_t i = 0; i < g_surs.size(); ++i)
    if (!g_surs[i].used) {
      g_surs[i] = S;
      *sid_out = (int32_t)i;
      return PDF_OK;
    }
  g_surs.push_back(S);
  *sid_out = (int32_t)(g_surs.size() - 1);
  return PDF_OK;
}

extern "C" int pdf_surrogate_destroy(int32_t sid) {
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  sur_release(*S);
  return PDF_OK;
}

extern "C" int pdf_surrogate_set_data(int32_t sid, const double* x, const double* q2, int64_t n,
                                      pdf_stream_t stream) {
  if (n < 16 || !x || !q2) return fail(PDF_ERR_ARG, "need >= 16 device training points");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  Member* M = sur_member(*S);
  if (!M) return fail(PDF_ERR_MEMBER, "surrogate's member %d was unloaded", S->member);
  hipStream_t s = (hipStream_t)stream;
  const int O = sur_out_width(), P = (int)M->pids.size();
  // the old set is released first; until the new one is complete, training finds no data
  sur_free_graph(*S);
  if (S->d_in) (void)hipFree(S->d_in);
  S->d_in = nullptr;
  S->d_t = nullptr;
  S->n_train = 0;
  // every sample: inputs, targets, in-domain flag; then the in-domain samples, in order
  void* tmp = nullptr;
  const size_t b_in = align_up((size_t)n * (2 + O) * 4, 256), b_xf = align_up((size_t)n * P * 8, 256);
  hipError_t e = hipMalloc(&tmp, b_in + b_xf + align_up((size_t)n, 256) + (size_t)n * 8);
  if (e != hipSuccess) return fail_hip(e, "hipMalloc(training samples)");
  float* in_all = static_cast<float*>(tmp);
  float* t_all = in_all + 2 * n;
  double* xf = reinterpret_cast<double*>(static_cast<unsigned char*>(tmp) + b_in);
  unsigned char* keep = static_cast<unsigned char*>(tmp) + b_in + b_xf;
  int64_t* idx = reinterpret_cast<int64_t*>(keep + align_up((size_t)n, 256));
  ReqCols rc{};
  build_req(*M, nullptr, 0, rc);
  // targets from this library's FP64 interpolator
  const LaunchCfg cfg{g_ncu, g_blocks_per_cu, g_vector_cols};
  e = launch_xfxq2_f64(M->dev, rc, x, q2, n, xf, g_nerr, lds_grid_elems(M->dev, false, n), M->invL01, cfg, nullptr,
                       nullptr, false, s);
  if (e == hipSuccess) e = sur_prep(S->sd, M->dev, x, q2, xf, n, in_all, t_all, keep, s);
  std::vector<unsigned char> hkeep((size_t)n);
  if (e == hipSuccess) e = hipMemcpyAsync(hkeep.data(), keep, (size_t)n, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  std::vector<int64_t> hidx;
  if (e == hipSuccess) {
    hidx.reserve((size_t)n);
    for (int64_t i = 0; i < n; ++i)
      if (hkeep[(size_t)i]) hidx.push_back(i);
  }
  const int64_t nk = (int64_t)hidx.size();
  float* din = nullptr;
  if (e == hipSuccess && nk < 16) {
    (void)hipFree(tmp);
    return fail(PDF_ERR_ARG, "only %lld of the %lld points lie in the network's domain (need >= 16)",
                (long long)nk, (long long)n);
  }
  if (e == hipSuccess) e = hipMemcpyAsync(idx, hidx.data(), (size_t)nk * 8, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMalloc(&din, (size_t)nk * (2 + O) * 4);
  if (e == hipSuccess) e = sur_gather(in_all, t_all, idx, nk, din, din + 2 * nk, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(tmp);
  if (e != hipSuccess) {
    if (din) (void)hipFree(din);
    return fail_hip(e, "surrogate targets");
  }
  S->d_in = din;
  S->d_t = din + 2 * nk;
  S->n_train = nk;
  return PDF_OK;
}

extern "C" int pdf_surrogate_train(int32_t sid, const pdf_train_opts* opts, pdf_stream_t stream) {
  if (!opts) return fail(PDF_ERR_ARG, "null opts");
  const int steps = opts->steps, batch = opts->batch;
  if (steps < 0 || batch < 16 || (batch & 15) || opts->total_steps < 1 || !(opts->lr >= 0.0f) ||
      !(opts->lr_final >= 0.0f))
    return fail(PDF_ERR_ARG, "bad training options");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  if (S->n_train < batch) return fail(PDF_ERR_STATE, "training data smaller than one batch (call set_data)");
  int rc = sur_ensure_batch(*S, batch);
  if (rc != PDF_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  const int64_t nb = S->n_train / batch;
  if (steps == 0) return PDF_OK;
  hipError_t e = sur_train_prepare();
  if (e != hipSuccess) return fail_hip(e, "surrogate training set-up");
  e = sur_train_begin(S->b, S->step, nb, batch, opts->total_steps, opts->lr, opts->lr_final, opts->loss_out, s);
  if (e != hipSuccess) return fail_hip(e, "surrogate training start");
  if (opts->use_graph) {
    if (S->g_batch != batch || S->g_in != S->d_in || S->g_bmem != S->bmem) sur_free_graph(*S);
    int left = steps;
    for (int k = 0; k < 2; ++k) {
      if (left < kGraphSteps[k]) continue;
      if (!S->exec[k] && (rc = sur_record_steps(*S, batch, k)) != PDF_OK) return rc;
      for (; left >= kGraphSteps[k]; left -= kGraphSteps[k])
        if ((e = hipGraphLaunch(S->exec[k], s)) != hipSuccess) return fail_hip(e, "hipGraphLaunch(training step)");
    }
  } else {
    for (int i = 0; i < steps; ++i)
      if ((e = sur_train_step(S->b, S->d_in, S->d_t, batch, s)) != hipSuccess)
        return fail_hip(e, "surrogate training step");
  }
  S->step += steps;
  return PDF_OK;
}

extern "C" int pdf_surrogate_grad(int32_t sid, const float* in, const float* target, int32_t batch, float* grad_out,
                                  float* loss_out, pdf_stream_t stream) {
  if (!in || !target || !grad_out || !loss_out || batch < 16 || (batch & 15))
    return fail(PDF_ERR_ARG, "bad gradient arguments");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  int rc = sur_ensure_batch(*S, batch);
  if (rc != PDF_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = sur_forward_backward(S->b, in, target, batch, loss_out, s);
  if (e == hipSuccess) e = hipMemcpyAsync(grad_out, S->b.G, (size_t)sur_nparams() * 4, hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return fail_hip(e, "surrogate gradient");
  return PDF_OK;
}

extern "C" int pdf_surrogate_adam(int32_t sid, const float* grad, float lr, pdf_stream_t stream) {
  if (!grad || !(lr >= 0.0f)) return fail(PDF_ERR_ARG, "bad Adam arguments");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(S->b.G, grad, (size_t)sur_nparams() * 4, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = sur_adam(S->b, lr, (int)(S->step + 1), s);
  if (e != hipSuccess) return fail_hip(e, "surrogate Adam step");
  ++S->step;
  return PDF_OK;
}

extern "C" int pdf_surrogate_params(int32_t sid, float* host, int32_t write) {
  if (!host) return fail(PDF_ERR_ARG, "null host buffer");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  const size_t nb = (size_t)sur_nparams() * 4;
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) {
    if (write) {
      e = hipMemcpy(S->b.P, host, nb, hipMemcpyHostToDevice);
      if (e == hipSuccess) e = sur_refresh_bf16(S->b, nullptr);
      if (e == hipSuccess) e = hipDeviceSynchronize();
    } else {
      e = hipMemcpy(host, S->b.P, nb, hipMemcpyDeviceToHost);
    }
  }
  if (e != hipSuccess) return fail_hip(e, "surrogate parameters");
  return PDF_OK;
}

extern "C" int pdf_surrogate_xfxq2(int32_t sid, const int32_t* pids, int32_t n_pids, const double* x,
                                   const double* q2, int64_t n, float* out, pdf_stream_t stream) {
  int rc = check_stream_args(x, q2, n);
  if (rc != PDF_OK) return rc;
  if (n > 0 && !out) return fail(PDF_ERR_ARG, "null out");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  Member* M = sur_member(*S);
  if (!M) return fail(PDF_ERR_MEMBER, "surrogate's member %d was unloaded", S->member);
  ReqCols cols{};
  if ((rc = build_req(*M, pids, n_pids, cols)) != PDF_OK) return rc;
  if (n == 0 || cols.n == 0) return PDF_OK;
  hipError_t e = sur_infer(S->sd, M->dev, cols, S->b, x, q2, n, out, M->invL01, g_nerr, g_ncu, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch surrogate inference");
  return PDF_OK;
}

extern "C" int pdf_surrogate_save(int32_t sid, const char* path) {
  if (!path) return fail(PDF_ERR_ARG, "null path");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  const int NP = sur_nparams();
  std::vector<float> buf((size_t)3 * NP);
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(buf.data(), S->b.P, (size_t)NP * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(buf.data() + NP, S->b.M, (size_t)NP * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(buf.data() + 2 * NP, S->b.V, (size_t)NP * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e, "surrogate save");
  const uint32_t version = 1, np = (uint32_t)NP;
  const int64_t step = S->step;
  uint64_t h = fnv1a(reinterpret_cast<const unsigned char*>(&step), 8);
  h = fnv1a(reinterpret_cast<const unsigned char*>(buf.data()), buf.size() * 4, h);
  FILE* f = fopen(path, "wb");
  if (!f) return fail(PDF_ERR_ARG, "cannot open %s for writing", path);
  bool ok = fwrite(kSurMagic, 1, 8, f) == 8 && fwrite(&version, 4, 1, f) == 1 && fwrite(&np, 4, 1, f) == 1 &&
            fwrite(&step, 8, 1, f) == 1 && fwrite(buf.data(), 4, buf.size(), f) == buf.size() &&
            fwrite(&h, 8, 1, f) == 1;
  ok = (fclose(f) == 0) && ok;
  if (!ok) return fail(PDF_ERR_ARG, "write to %s failed", path);
  return PDF_OK;
}

extern "C" int pdf_surrogate_load(int32_t sid, const char* path) {
  if (!path) return fail(PDF_ERR_ARG, "null path");
  std::lock_guard<std::mutex> lock(g_mu);
  Surrogate* S = get_sur(sid);
  if (!S) return fail(PDF_ERR_ARG, "unknown surrogate %d", sid);
  const int NP = sur_nparams();
  FILE* f = fopen(path, "rb");
  if (!f) return fail(PDF_ERR_ARG, "cannot open %s", path);
  char mg[8];
  uint32_t version = 0, np = 0;
  int64_t step = 0;
  uint64_t h = 0;
  std::vector<float> buf((size_t)3 * NP);
  bool ok = fread(mg, 1, 8, f) == 8 && fread(&version, 4, 1, f) == 1 && fread(&np, 4, 1, f) == 1;
  ok = ok && std::memcmp(mg, kSurMagic, 8) == 0 && version == 1 && np == (uint32_t)NP;
  ok = ok && fread(&step, 8, 1, f) == 1 && fread(buf.data(), 4, buf.size(), f) == buf.size() &&
       fread(&h, 8, 1, f) == 1;
  fclose(f);
  if (!ok) return fail(PDF_ERR_ARG, "%s is not a surrogate checkpoint of this layout", path);
  uint64_t h2 = fnv1a(reinterpret_cast<const unsigned char*>(&step), 8);
  h2 = fnv1a(reinterpret_cast<const unsigned char*>(buf.data()), buf.size() * 4, h2);
  if (h2 != h) return fail(PDF_ERR_ARG, "%s: checksum mismatch", path);
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(S->b.P, buf.data(), (size_t)NP * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(S->b.M, buf.data() + NP, (size_t)NP * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(S->b.V, buf.data() + 2 * NP, (size_t)NP * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = sur_refresh_bf16(S->b, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return fail_hip(e, "surrogate load");
  S->step = step;
  return PDF_OK;
}

extern "C" int pdf_mc_workspace_bytes(int64_t n, int64_t* bytes_out) {
  if (!bytes_out || n < 0) return fail(PDF_ERR_ARG, "bad argument");
  *bytes_out = (n == 0 ? 1 : mc_partials(n)) * (int64_t)sizeof(double);
  return PDF_OK;
}

template <typename T>
static int mc_sum_impl(const T* xf1, const T* xf2, int32_t n_pids, const double* alphas, int64_t n, double* workspace,
                       double* sum_out, pdf_stream_t stream) {
  if (n < 0 || n_pids < 1 || n_pids > kMaxReq) return fail(PDF_ERR_ARG, "bad n or n_pids");
  if (!sum_out || !workspace) return fail(PDF_ERR_ARG, "null output or workspace");
  if (n > 0 && (!xf1 || !xf2 || !alphas)) return fail(PDF_ERR_ARG, "null input");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  hipError_t e = launch_mc_sum<T>(xf1, xf2, n_pids, alphas, n, workspace, sum_out, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch mc sum");
  return PDF_OK;
}

extern "C" int pdf_mc_chunk_sum(const double* xf1, const double* xf2, int32_t n_pids, const double* alphas, int64_t n,
                                double* workspace, double* sum_out, pdf_stream_t stream) {
  return mc_sum_impl<double>(xf1, xf2, n_pids, alphas, n, workspace, sum_out, stream);
}

extern "C" int pdf_mc_chunk_sum_f32(const float* xf1, const float* xf2, int32_t n_pids, const double* alphas,
                                    int64_t n, double* workspace, double* sum_out, pdf_stream_t stream) {
  return mc_sum_impl<float>(xf1, xf2, n_pids, alphas, n, workspace, sum_out, stream);
}

// LDS of the one-kernel form besides the tables: the summation tree and the request's column lists.
constexpr size_t kMcFixedBytes = 1024 * 8 + (2 * kMaxReq + kMaxSub + 4) * 4;

template <typename T>
static int mc_fused_impl(int32_t member, const int32_t* pids, int32_t n_pids, const double* x1, const double* x2,
                         const double* q2, int64_t n, double* workspace, double* sum_out, pdf_stream_t stream) {
  if (n < 0) return fail(PDF_ERR_ARG, "n < 0");
  if (!sum_out || !workspace) return fail(PDF_ERR_ARG, "null output or workspace");
  if (n > 0 && (!x1 || !x2 || !q2)) return fail(PDF_ERR_ARG, "null input");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  Member* M = get_member(member);
  if (!M) return fail(PDF_ERR_MEMBER, "unknown member %d", member);
  if (!g_has_alphas) return fail(PDF_ERR_STATE, "no alpha_s table loaded");
  ReqCols rcols{};
  if ((rc = build_req(*M, pids, n_pids, rcols)) != PDF_OK) return rc;
  if (M->mc_bytes + g_alphas_mc_bytes + kMcFixedBytes > kLdsBytes)
    return fail(PDF_ERR_GRID, "location tables too large for the fused kernel; use pdf_xfxq2 + pdf_mc_chunk_sum");
  hipError_t e = launch_mc_fused<T>(M->dev, rcols, g_alphas, x1, x2, q2, n, workspace, sum_out, g_nerr, M->invL01,
                                    g_ncu, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch fused mc sum");
  return PDF_OK;
}

extern "C" int pdf_mc_fused(int32_t member, const int32_t* pids, int32_t n_pids, const double* x1, const double* x2,
                            const double* q2, int64_t n, double* workspace, double* sum_out, pdf_stream_t stream) {
  return mc_fused_impl<double>(member, pids, n_pids, x1, x2, q2, n, workspace, sum_out, stream);
}

extern "C" int pdf_mc_fused_f32(int32_t member, const int32_t* pids, int32_t n_pids, const double* x1,
                                const double* x2, const double* q2, int64_t n, double* workspace, double* sum_out,
                                pdf_stream_t stream) {
  return mc_fused_impl<float>(member, pids, n_pids, x1, x2, q2, n, workspace, sum_out, stream);
}

extern "C" int pdf_fk_contract(const double* pdf, const double* fk, int32_t nrep, int32_t ndat, int64_t K,
                               double* out, pdf_stream_t stream) {
  if (nrep < 0 || ndat < 0 || K < 0) return fail(PDF_ERR_ARG, "negative size");
  if (nrep > (1 << 22)) return fail(PDF_ERR_ARG, "nrep above 4194304");
  if (nrep > 0 && ndat > 0 && (!out || (K > 0 && (!pdf || !fk)))) return fail(PDF_ERR_ARG, "null device pointer");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_init();
  if (rc != PDF_OK) return rc;
  if (nrep == 0 || ndat == 0) return PDF_OK;
  const int S = fk_slices(nrep, ndat, K, g_ncu);
  const size_t need = S > 1 ? (size_t)S * nrep * ndat * sizeof(double) : 0;
  if (need > g_fk_ws_bytes) {
    // the stream's earlier work may still read the old buffer
    hipError_t e = g_fk_ws ? hipStreamSynchronize((hipStream_t)stream) : hipSuccess;
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
    if (g_fk_ws) (void)hipFree(g_fk_ws);
    g_fk_ws = nullptr;
    g_fk_ws_bytes = 0;
    e = hipMalloc(&g_fk_ws, need);
    if (e != hipSuccess) return fail_hip(e, "hipMalloc(fk workspace)");
    g_fk_ws_bytes = need;
  }
  hipError_t e = launch_fk_contract(pdf, fk, nrep, ndat, K, out, S, static_cast<double*>(g_fk_ws),
                                    (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch fk contraction");
  return PDF_OK;
}

extern "C" int pdf_fk_contract_noalloc(const double* pdf, const double* fk, int32_t nrep, int32_t ndat, int64_t K,
                                       double* out, pdf_stream_t stream) {
  if (nrep < 0 || ndat < 0 || K < 0) return fail(PDF_ERR_ARG, "negative size");
  if (nrep > (1 << 22)) return fail(PDF_ERR_ARG, "nrep above 4194304");
  if (nrep > 0 && ndat > 0 && (!out || (K > 0 && (!pdf || !fk)))) return fail(PDF_ERR_ARG, "null device pointer");
  std::lock_guard<std::mutex> lock(g_mu);
  int rc = ensure_device();
  if (rc != PDF_OK) return rc;
  if (nrep == 0 || ndat == 0) return PDF_OK;
  const int L = fk_limit_slices(nrep, ndat, K, g_ncu);
  const size_t need = L > 1 ? (size_t)L * nrep * ndat * sizeof(double) : 0;
  if (need > fk_scratch_bytes())
    return fail(PDF_ERR_ARG, "partial sums of %d K slices x %d x %d doubles need %zu bytes, above the %zu-byte scratch",
                L, nrep, ndat, need, fk_scratch_bytes());
  const int S = fk_slices(nrep, ndat, K, g_ncu);  // its partial sums always fit
  // every partial sum is written by the contraction kernel before the reduction reads it: nothing to clear
  hipError_t e = launch_fk_contract(pdf, fk, nrep, ndat, K, out, S, g_fk_scratch, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e, "launch fk contraction");
  return PDF_OK;
}

extern "C" int pdf_set_lds_policy(int32_t policy) {
  if (policy < 0 || policy > 2) return fail(PDF_ERR_ARG, "policy must be 0, 1 or 2");
  std::lock_guard<std::mutex> lock(g_mu);
  g_lds_policy = policy;
  return PDF_OK;
}

extern "C" const char* pdf_last_error(void) { return g_err.c_str(); }

extern "C" int pdf_shutdown(void) {
  std::lock_guard<std::mutex> lock(g_mu);
  for (auto& M : g_members)
    if (M.used && M.dmem) {
      (void)hipFree(M.dmem);
      for (Layout& l : M.layouts) layout_release(l);
    }
  g_members.clear();

  if (g_alphas_mem) (void)hipFree(g_alphas_mem);
  g_alphas_mem = nullptr;
  g_has_alphas = false;
  for (auto& P : g_plans)
    if (P.used) plan_release(P);
  g_plans.clear();
  for (auto& S : g_surs)
    if (S.used) sur_release(S);
  g_surs.clear();
  if (g_runs.dev) (void)hipFree(g_runs.dev);
  if (g_runs.host) (void)hipHostFree(g_runs.host);
  g_runs = RunPool();
  if (g_nerr) (void)hipFree(g_nerr);
  g_nerr = nullptr;
  if (g_fk_ws) (void)hipFree(g_fk_ws);
  g_fk_ws = nullptr;
  g_fk_ws_bytes = 0;
  g_fk_scratch = nullptr;  // the array itself stays with the process
  g_dev_ready = false;
  g_init = false;
  return PDF_OK;
}
