// FastKernel-style contraction of PDF members with a kernel table (paper
// section 4.3: theory predictions are convolutions of FK tables with PDFs
// evaluated on an x grid; the multi-member form evaluates many replicas at
// once):
//   T[r][d] = sum_k F[r][k] * FK[d][k],   k = (x point i, flavour a) flattened,
// a dense FP64 contraction of the replica matrix F [nrep][K] with the table
// [ndat][K], on the FP64 matrix cores (v_mfma_f64_16x16x4_f64).
//
// Two kernels: k_fk_contract for one tile of members (up to 112), k_fk_tiles
// for more and for the largest tables (see fk_staged).  The summation order is fixed by the sizes and the number of
// compute units (deterministic results).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pdfmi_dev.h"

namespace pdfmi {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kFkBN = 32;            // table rows of a tile
constexpr int kFkWaves = 4;          // ranges of k per workgroup
constexpr int kFkThreads = 64 * kFkWaves;
constexpr int kFkStep = 16;          // k per register set
constexpr int kFkMaxMT = 7;

typedef double f64x2 __attribute__((ext_vector_type(2)));

// 2 consecutive doubles at 8-byte alignment (rows of odd length)
__device__ __forceinline__ f64x2 load2(const double* p) {
  f64x2 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

// Up to 112 members.  The table is read once and the matrix cores need few
// operands (an instruction keeps a SIMD's busy for 64 clocks), so what cost the
// time were padding, barriers and the slices' partial sums.  Hence no LDS and
// no barrier in the loop: a wave computes 16 MT members x 32 table rows over its
// own range of k, every operand loaded straight into registers.  The k of an
// instruction may be any four, as long as both operands agree: lane (r, q)
// takes k0 + 8 j + 2 q and + 1, so a load is 16 bytes per lane and 64
// contiguous bytes per row.  The four waves of a workgroup take four ranges of
// k of one tile and add their sums through LDS at the end, which leaves few
// slices to add in global memory.  K = 31395, 1024 table rows: 10 members 59-63 us
// (staged tiles of 64 or 80 x 128: 101), 30: 79 (104), 50: 99 (108), 80: 122
// (130), 100: 144 (164); 100 rows x 100 members 42 (65).  400 members took 496
// us here and 456 with the staged tiles, whose operands eight waves share.
// Rows beyond the last are read as the last and not stored; k beyond the last
// reads as zero.
//
// One (16 MT x 32 tile, K slice) per workgroup: sums over
// [slice * 4 * kwave, min(K, (slice + 1) * 4 * kwave)) to T + slice * nrep * ndat.
template <int MT>
__global__ __launch_bounds__(kFkThreads) void k_fk_contract(const double* __restrict__ F,
                                                            const double* __restrict__ FK, int nrep, int ndat,
                                                            int64_t K, int64_t kwave, int ntiles, int S,
                                                            double* __restrict__ T) {
  extern __shared__ __align__(16) double sums[];  // [wave][MT * 2 * 4][64]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kq = lane >> 4;
  // workgroups go round the 8 XCDs by index: each XCD takes a contiguous run of
  // (slice, n tile), so that the tiles that read one piece of F share an L2
  const int work = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (work >= S * ntiles) return;
  const int slice = work / ntiles, n0 = (work - slice * ntiles) * kFkBN;
  const int64_t kbeg = min(K, ((int64_t)slice * kFkWaves + wave) * kwave), kend = min(K, kbeg + kwave);
  const double* pa[MT];
  const double* pb[2];
#pragma unroll
  for (int t = 0; t < MT; ++t) pa[t] = F + (int64_t)min(16 * t + r16, nrep - 1) * K + 2 * kq;
#pragma unroll
  for (int c = 0; c < 2; ++c) pb[c] = FK + (int64_t)min(n0 + 16 * c + r16, ndat - 1) * K + 2 * kq;
  f64x4 acc[MT][2];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t][0] = acc[t][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  // registers of the steps in flight: the table's operands four steps ahead
  // (they come from HBM), F's one step (they come from L2)
  f64x2 b[4][2][2], a[2][2][MT];
  auto fetch_b = [&](f64x2 (&d)[2][2], int64_t k0) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < 2; ++j) d[j][c] = load2(pb[c] + k0 + 8 * j);
  };
  auto fetch_a = [&](f64x2 (&d)[2][MT], int64_t k0) {
#pragma unroll
    for (int t = 0; t < MT; ++t)  // both halves of a 128-byte piece of a row one after the other
#pragma unroll
      for (int j = 0; j < 2; ++j) d[j][t] = load2(pa[t] + k0 + 8 * j);
  };
  auto multiply = [&](const f64x2 (&sa)[2][MT], const f64x2 (&sb)[2][2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[j][t][e], sb[j][c][e], acc[t][c], 0, 0, 0);
  };
  const int64_t steps = (kend - kbeg) / kFkStep;  // whole steps
  if (steps > 0) {
    // step i of the range, clamped to its last (in bounds, unused past it)
    auto at = [&](int64_t i) { return kbeg + min(i, steps - 1) * kFkStep; };
#pragma unroll
    for (int i = 0; i < 4; ++i) fetch_b(b[i], at(i));
    fetch_a(a[0], at(0));
    int64_t i = 0;
    for (; i + 4 <= steps; i += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        fetch_a(a[(u + 1) & 1], at(i + u + 1));
        __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products of the other set
        multiply(a[u & 1], b[u]);
        fetch_b(b[u], at(i + u + 4));
      }
    const int left = (int)(steps - i);  // 0..3
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u < left) {
        fetch_a(a[(u + 1) & 1], at(i + u + 1));
        multiply(a[u & 1], b[u]);
      }
  }
  if (kbeg + steps * kFkStep < kend) {  // the last k of all, one by one
    const int64_t k0 = kbeg + steps * kFkStep;
    auto one = [&](const double* p, int64_t k) { return k + 2 * kq < kend ? p[k] : 0.0; };
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
#pragma unroll
        for (int c = 0; c < 2; ++c) b[0][j][c][e] = one(pb[c], k0 + 8 * j + e);
#pragma unroll
        for (int t = 0; t < MT; ++t) a[0][j][t][e] = one(pa[t], k0 + 8 * j + e);
      }
    multiply(a[0], b[0]);
  }
  // the waves' sums, in wave order; each wave adds and stores a quarter
  constexpr int kVals = MT * 2 * 4;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) sums[(wave * kVals + (t * 2 + c) * 4 + v) * 64 + lane] = acc[t][c][v];
  __syncthreads();
  T += (int64_t)slice * nrep * ndat;
  for (int e = wave; e < kVals; e += kFkWaves) {
    double x = sums[e * 64 + lane];
#pragma unroll
    for (int w = 1; w < kFkWaves; ++w) x += sums[(w * kVals + e) * 64 + lane];
    // accumulator layout of the FP64 16x16x4 form: value v of a lane is row
    // lane / 16 + 4 v, column lane % 16
    const int m = (e >> 3) * 16 + kq + 4 * (e & 3), n = n0 + ((e >> 2) & 1) * 16 + r16;
    if (m < nrep && n < ndat) T[(int64_t)m * ndat + n] = x;
  }
}

constexpr int kFkTileN = 128, kFkBK = 32, kFkLd = kFkBK + 1, kFkTileThreads = 512;
constexpr int kFkSlotsPerCu = 2;  // resident workgroups per compute unit (LDS and the 128-VGPR bound)

// More members.  Tiling: a workgroup of 8 waves computes a BM x 128 tile of T (BM = 64 or
// 80 members, whichever pads the member count less, x 128 table rows); wave w
// owns table rows 16 w .. 16 w + 15 of the tile against all BM members, as
// BM / 16 MFMA tiles of 16 x 16 sharing one B operand per k step.  The kernel
// is held to 128 VGPRs so two workgroups share a compute unit (4 waves per
// SIMD).
// K is walked in steps of 32 staged in LDS as rows of 33 doubles, with the
// next step's global loads (32 consecutive k per half-wave: 256-byte
// segments; one pointer per operand advanced by 32 each step, row i of a
// thread 16 i K further) issued before the current step's MFMAs.  An operand
// read (lane = row r + 16 k-column q) is served 16 lanes (128 bytes) at a
// time; with a row stride of 33 doubles the 16 rows of one q land on 16
// distinct 8-byte bank slots (a stride of 36 put rows r and r + 8 on the
// same slot and cost ~45 % of the kernel's cycles in bank conflicts).
// Out-of-range rows and k read as zero.  K is split into S slices whose
// partial sums are added in slice order, so the summation order is fixed
// (deterministic results); S is chosen from the sizes and the number of
// compute units only, to fill the two workgroup slots of every compute unit
// evenly (a launch of 520 workgroups on 512 slots ran 25 % slower than one of
// 480).
//
// One (BM x 128 tile, K slice) per workgroup, BM = 16 MT: the slice
// [blockIdx.z * kslice, min(K, (blockIdx.z + 1) * kslice)) of the sum goes to
// T + blockIdx.z * nrep * ndat (the partial sums of the slices are added in
// slice order by k_fk_reduce).
template <int MT>
__global__ __launch_bounds__(kFkTileThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_fk_tiles(
    const double* __restrict__ F, const double* __restrict__ FK, int nrep, int ndat, int64_t K, int64_t kslice,
    double* __restrict__ T) {
  constexpr int BM = 16 * MT;
  constexpr int kRowsA = BM * kFkBK / kFkTileThreads, kRowsB = kFkTileN * kFkBK / kFkTileThreads;  // loads per thread
  __shared__ double sa[BM * kFkLd];
  __shared__ double sb[kFkTileN * kFkLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * kFkTileN;
  // cooperative loads: thread -> k = tid % 32 of rows tid / 32 + 16 i
  const int lk = tid & 31, lr = tid >> 5;
  const int64_t kbeg = (int64_t)blockIdx.z * kslice, kend = min(K, kbeg + kslice);
  T += (int64_t)blockIdx.z * nrep * ndat;
  const double* pa = F + (int64_t)(m0 + lr) * K + kbeg + lk;
  const double* pb = FK + (int64_t)(n0 + lr) * K + kbeg + lk;
  const int64_t rs = 16 * K;                             // 16 rows further
  const int na = nrep - m0 - lr, nb = ndat - n0 - lr;  // row i of the thread exists when 16 i < na (nb)
  int64_t krem = kend - kbeg - lk;                       // its k exists while krem > 0
  double ra[kRowsA], rb[kRowsB];
  auto fetch = [&]() {
    const bool kok = krem > 0;
#pragma unroll
    for (int i = 0; i < kRowsA; ++i) ra[i] = (kok && 16 * i < na) ? pa[i * rs] : 0.0;
#pragma unroll
    for (int i = 0; i < kRowsB; ++i) rb[i] = (kok && 16 * i < nb) ? pb[i * rs] : 0.0;
    pa += kFkBK;
    pb += kFkBK;
    krem -= kFkBK;
  };
  f64x4 acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int r16 = lane & 15, kq = lane >> 4;
  fetch();
  for (int64_t k0 = kbeg; k0 < kend; k0 += kFkBK) {
    __syncthreads();  // previous step's operands consumed
#pragma unroll
    for (int i = 0; i < kRowsA; ++i) sa[(lr + 16 * i) * kFkLd + lk] = ra[i];
#pragma unroll
    for (int i = 0; i < kRowsB; ++i) sb[(lr + 16 * i) * kFkLd + lk] = rb[i];
    __syncthreads();
    if (k0 + kFkBK < kend) fetch();
#pragma unroll
    for (int kk = 0; kk < kFkBK; kk += 4) {
      const double b = sb[(wave * 16 + r16) * kFkLd + kk + kq];  // B: column r16, k = kq
      double a[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) a[t] = sa[(t * 16 + r16) * kFkLd + kk + kq];  // A: row r16, k = kq
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b, acc[t], 0, 0, 0);
    }
  }
  // accumulator layout of the FP64 16x16x4 form: value v of a lane is row
  // lane / 16 + 4 v, column lane % 16
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = m0 + t * 16 + kq + 4 * v;
      const int n = n0 + wave * 16 + r16;
      if (m < nrep && n < ndat) T[(int64_t)m * ndat + n] = acc[t][v];
    }
}

// T[m][n] = sum over slices s = 0..S-1 (in that order) of P[s][m][n].
__global__ void k_fk_reduce(const double* __restrict__ P, int S, int64_t mn, double* __restrict__ T) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < mn; i += (int64_t)gridDim.x * blockDim.x) {
    double acc = P[i];
    for (int s = 1; s < S; ++s) acc += P[(int64_t)s * mn + i];
    T[i] = acc;
  }
}

// k_fk_contract takes up to this many members.
constexpr int kFkOneTile = 16 * kFkMaxMT;

// Is the contraction one for k_fk_tiles?  Above 112 members always.  Up to 80,
// where its one tile of members pads little, also for tables beyond 256 MB (the
// last cache): k_fk_contract then reads F from L2 four times as often as the
// tiles of 128 table rows do, and rows that do not start on a 128-byte line
// cost it more.  Times of k_fk_contract in those of k_fk_tiles, by members,
// warm and with a new table each time: 1024 rows x 8001 0.64-0.76 and 0.72-0.94;
// 1024 x 31395 24: 0.66, 32: 0.82 and 0.95, 64: 0.94 and 1.04; 3000 x 16001 24:
// 1.01, 32: 1.07, 64: 1.29 and 1.21; 700 x 60001 33: 0.80, 64: 0.98; 10000 x 31395 24: 1.09, 32: 1.17, 64: 1.34,
// 80: 1.25; with rows on lines (31392) 32: 0.92, 48: 1.05, 64: 1.11.  At 81 to
// 112 members 0.6-1.03 everywhere (two tiles there).
static bool fk_staged(int nrep, int ndat, int64_t K) {
  if (nrep > kFkOneTile) return true;
  const bool lines = K % 16 == 0;
  const int64_t least = nrep > 48 ? 33000000 : 45000000;  // values of the table
  return nrep <= 80 && nrep > (lines ? 48 : 24) && K >= least / std::max(ndat, 1);
}

// Rows per member tile of k_fk_tiles: 80 when that pads the member count no
// more than 64 does (400 members: 5 tiles of 80 against 7 of 64), else 64.
static int fk_tile_rows(int nrep) {
  const int64_t p64 = (int64_t)(nrep + 63) / 64 * 64, p80 = (int64_t)(nrep + 79) / 80 * 80;
  return p80 <= p64 ? 80 : 64;
}

constexpr size_t kFkScratchBytes = (size_t)64 << 20;

// The smallest S <= smax whose tiles x S workgroups fill at least 93 % of the
// rounds of workgroup slots they occupy; failing that the S with the fullest
// rounds.  Extra slices cost partial sums written and added.
static int fk_fill(int64_t tiles, int64_t slots, int64_t smax) {
  int best = 1;
  double best_fill = -1.0;
  for (int64_t S = 1; S <= smax; ++S) {
    const int64_t wg = tiles * S;
    const double fill = (double)wg / (double)(((wg + slots - 1) / slots) * slots);
    if (fill >= 0.93) return (int)S;
    if (fill > best_fill + 1e-12) {
      best_fill = fill;
      best = (int)S;
    }
  }
  return best;
}

// K slices of k_fk_tiles, which pdf_fk_contract_noalloc also counts when it
// decides whether a contraction is within its scratch: two workgroups per
// compute unit, at least 8 K steps each, at most 64 slices.
int fk_limit_slices(int nrep, int ndat, int64_t K, int n_cu) {
  const int bm = fk_tile_rows(nrep);
  return fk_fill((int64_t)((ndat + kFkTileN - 1) / kFkTileN) * ((nrep + bm - 1) / bm),
                 (int64_t)kFkSlotsPerCu * std::max(n_cu, 1),
                 std::max<int64_t>(1, std::min<int64_t>(64, K / (8 * kFkBK))));
}

// K slices of a contraction.  With k_fk_contract: workgroups of four waves, one per
// compute unit for tiles of 64 members or more (its registers then hold one
// wave per SIMD), else two; at least 64 k per wave, partial sums within the
// scratch size.
int fk_slices(int nrep, int ndat, int64_t K, int n_cu) {
  if (fk_staged(nrep, ndat, K)) return fk_limit_slices(nrep, ndat, K, n_cu);
  const int64_t fit = (int64_t)(kFkScratchBytes / 8) / std::max<int64_t>(1, (int64_t)nrep * ndat);
  return fk_fill((ndat + kFkBN - 1) / kFkBN, (int64_t)(nrep > 48 ? 1 : 2) * std::max(n_cu, 1),
                 std::max<int64_t>(1, std::min({(int64_t)64, K / (64 * kFkWaves), fit})));
}

// Partial sums of the K slices for callers that cannot allocate
// (pdf_fk_contract_noalloc): a fixed array in device memory, one per GPU the
// library runs on, held until the process ends.  Host code never passes the
// array's name to a kernel: fk_scratch_setup looks up its device address once
// per device and the launches take that pointer.
static __device__ __align__(256) double scratch[kFkScratchBytes / sizeof(double)];

constexpr int kFkMaxDevices = 64;
static double* g_scratch_ptr[kFkMaxDevices] = {};

size_t fk_scratch_bytes() { return kFkScratchBytes; }

// Device address of the scratch array on `device`, which must be the current
// device; looked up on the first call for that device.
hipError_t fk_scratch_setup(int device, double** out) {
  *out = nullptr;
  if (device < 0 || device >= kFkMaxDevices) return hipErrorInvalidDevice;
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

template <int MT>
static hipError_t launch_tiles(const double* F, const double* FK, int nrep, int ndat, int64_t K, int S, double* dst,
                               hipStream_t s) {
  const int ntiles = (ndat + kFkBN - 1) / kFkBN;
  const int64_t work = (int64_t)ntiles * S;
  const int64_t per = (K + (int64_t)S * kFkWaves - 1) / ((int64_t)S * kFkWaves);
  const int64_t kwave = std::max<int64_t>(1, (per + kFkStep - 1) / kFkStep * kFkStep);
  if (work > 0x7ffffff0) return hipErrorInvalidValue;
  const size_t shm = sizeof(double) * kFkWaves * MT * 2 * 4 * 64;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&k_fk_contract<MT>), shm);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fk_contract<MT>, dim3((unsigned)((work + 7) / 8 * 8)), dim3(kFkThreads), shm, s, F, FK, nrep,
                     ndat, K, kwave, ntiles, S, dst);
  return hipGetLastError();
}

// ws: S * nrep * ndat doubles when S > 1 (unused otherwise).
hipError_t launch_fk_contract(const double* F, const double* FK, int nrep, int ndat, int64_t K, double* T, int S,
                              double* ws, hipStream_t s) {
  double* dst = S > 1 ? ws : T;
  hipError_t e = hipSuccess;
  if (fk_staged(nrep, ndat, K)) {
    int64_t kslice = (K + S - 1) / S;
    kslice = std::max<int64_t>((kslice + kFkBK - 1) / kFkBK * kFkBK, 1);
    const int bm = fk_tile_rows(nrep);
    const dim3 grid((unsigned)((ndat + kFkTileN - 1) / kFkTileN), (unsigned)((nrep + bm - 1) / bm), (unsigned)S);
    if (bm == 80)
      hipLaunchKernelGGL(k_fk_tiles<5>, grid, dim3(kFkTileThreads), 0, s, F, FK, nrep, ndat, K, kslice, dst);
    else
      hipLaunchKernelGGL(k_fk_tiles<4>, grid, dim3(kFkTileThreads), 0, s, F, FK, nrep, ndat, K, kslice, dst);
    e = hipGetLastError();
  } else switch ((nrep + 15) / 16) {
    case 1: e = launch_tiles<1>(F, FK, nrep, ndat, K, S, dst, s); break;
    case 2: e = launch_tiles<2>(F, FK, nrep, ndat, K, S, dst, s); break;
    case 3: e = launch_tiles<3>(F, FK, nrep, ndat, K, S, dst, s); break;
    case 4: e = launch_tiles<4>(F, FK, nrep, ndat, K, S, dst, s); break;
    case 5: e = launch_tiles<5>(F, FK, nrep, ndat, K, S, dst, s); break;
    case 6: e = launch_tiles<6>(F, FK, nrep, ndat, K, S, dst, s); break;
    default: e = launch_tiles<7>(F, FK, nrep, ndat, K, S, dst, s); break;
  }
  if (e != hipSuccess) return e;
  if (S > 1) {
    const int64_t mn = (int64_t)nrep * ndat;
    const int64_t nb = std::min<int64_t>((mn + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fk_reduce, dim3((unsigned)nb), dim3(256), 0, s, ws, S, mn, T);
  }
  return hipGetLastError();
}

}  // namespace pdfmi
