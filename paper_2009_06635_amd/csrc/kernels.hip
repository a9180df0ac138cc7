// HIP kernels for gfx950: x*f(x,Q^2) log-bicubic interpolation, point
// location, and alpha_s(Q^2) log-cubic interpolation.
//
// Interpolation (paper section 2.2): cubic Hermite in ln x then in ln Q^2 with
// finite-difference slopes, written as a separable 4x4 weighted sum
//   xf = sum_b v_b * sum_a w_a * f[sx+a][sq+b][col]
// where w (x direction) and v (Q^2 direction) are the Hermite weights of the
// point's cell, re-based onto a 4-knot stencil that stays inside the sub-grid
// (one-sided slopes at sub-grid edges give zero weight outside it).
// Extrapolation (figure 1 EXTRAPOLATE) uses anchor values on the edge rows or
// columns of the same stencil, combined in FP64.
//
// Work split: each wave takes its own tiles of 64 points (8 to 32 in small
// calls), with no workgroup barrier after the tables are staged.
//   phase 1, one lane per point: validate, region, one FP64 knot search per
//     axis (raw FP64 comparisons, all Q^2 sub-grids in one table), logarithms
//     by table, Hermite weights -> the wave's records in LDS;
//   phase 2, one lane per (point, flavour), or per (point, group of columns of
//     up to 16 bytes) where the request is every stored column in order or has
//     a compacted copy; consecutive lanes on consecutive output elements
//     (coalesced point-major stores): 16 grid reads from LDS (grid staged once
//     per workgroup when it fits) or from L2-resident global memory, 20 FMAs
//     per value.  Points outside the grid wait in a list until they fill a pass.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "interp_dev.h"
#include "layouts.h"
#include "tiles.h"
#include "pdfmi_dev.h"

namespace pdfmi {


// 16-byte column groups of the vectorised path.
template <typename T, int G>
struct VecOf;
template <>
struct VecOf<double, 2> { using type = double2; };
template <>
struct VecOf<float, 4> { using type = float4; };
template <>
struct VecOf<float, 2> { using type = float2; };
template <>
struct VecOf<double, 1> { using type = double; };
template <>
struct VecOf<float, 1> { using type = float; };

// Buffer resource over [base, base + bytes): loads and stores through it take
// a 32-bit per-lane byte offset plus a uniform (scalar) byte offset, so the
// stencil gathers need no 64-bit address arithmetic; the hardware returns
// zero for loads past `bytes` and drops stores past it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// G consecutive elements of T (G * sizeof(T) in {4, 8, 16} bytes).
template <typename T, int G>
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff, T* dst) {
  constexpr int kBytes = G * (int)sizeof(T);
  if constexpr (kBytes == 16) {
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    const unsigned int u[4] = {q.x, q.y, q.z, q.w};
    __builtin_memcpy(dst, u, 16);
  } else if constexpr (kBytes == 8) {
    const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    const unsigned int u[2] = {q.x, q.y};
    __builtin_memcpy(dst, u, 8);
  } else {
    static_assert(kBytes == 4, "unsupported gather width");
    const unsigned int u = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
    __builtin_memcpy(dst, &u, 4);
  }
}

// Cache policy of the output stores: 0 (default) or kStoreStream, the
// non-temporal hint.  While the grid is gathered through L2, the streamed
// output rows then displace fewer grid lines (measured 5-9 % faster for 1e7
// points); with the grid staged in LDS the hint made the same call slower
// (0.31 -> 0.55 ms in FP32), so those kernels keep the default.
constexpr int kStoreStream = 2;

template <typename T, int G, int kPolicy = 0>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, int voff, const T* src) {
  constexpr int kBytes = G * (int)sizeof(T);
  if constexpr (kBytes == 16) {
    unsigned int u[4];
    __builtin_memcpy(u, src, 16);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{u[0], u[1], u[2], u[3]}, r, voff, 0, kPolicy);
  } else if constexpr (kBytes == 8) {
    unsigned int u[2];
    __builtin_memcpy(u, src, 8);
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{u[0], u[1]}, r, voff, 0, kPolicy);
  } else {
    static_assert(kBytes == 4, "unsupported store width");
    unsigned int u;
    __builtin_memcpy(&u, src, 4);
    __builtin_amdgcn_raw_buffer_store_b32(u, r, voff, 0, kPolicy);
  }
}

// Workgroup copy of `bytes` (a multiple of 4; both pointers 16-byte
// aligned) from global memory to LDS.  Each thread issues eight 16-byte loads
// before it stores them: a loop of dependent load-store pairs waits out the
// memory latency once per element (a 72 KB grid: 18 round trips per thread).
template <int BS>
__device__ __forceinline__ void stage_copy(void* dst, const void* src, int64_t bytes) {
  const PDFMI_GLOBAL u32x4* s = (const PDFMI_GLOBAL u32x4*)src;
  u32x4* d = static_cast<u32x4*>(dst);
  const int64_t nv = bytes >> 4;
  for (int64_t i0 = threadIdx.x; i0 < nv; i0 += 8 * BS) {
    u32x4 r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = s[min(i0 + k * BS, nv - 1)];  // clamped: every load in bounds
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i0 + k * BS < nv) d[i0 + k * BS] = r[k];
  }
  const int tail = (int)((bytes & 15) >> 2);  // trailing 4-byte words
  if ((int)threadIdx.x < tail)
    reinterpret_cast<unsigned*>(d + nv)[threadIdx.x] = ((const PDFMI_GLOBAL unsigned*)(s + nv))[threadIdx.x];
}

// Workgroup copy of chosen columns of `rows` grid rows (global, P columns in a
// stride of Ps floats) into LDS rows of kRow floats: column c to position
// pos[c] (uniform; -1: not requested).  A thread takes whole rows, two at a
// time, in 16-byte loads.
template <int BS, int kRow>
__device__ __forceinline__ void stage_columns(float* dst, const float* src, int rows, int P, int Ps,
                                              const int* __restrict__ pos) {
  for (int c0 = 0; c0 < P; c0 += 12)
    for (int r0 = threadIdx.x; r0 < rows; r0 += 2 * BS) {
      const int r1 = min(r0 + BS, rows - 1);  // clamped: every access in bounds (the last row may be written twice)
      f32x4 q[2][3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (c0 + 4 * k < P) {
          q[0][k] = *(const PDFMI_GLOBAL f32x4*)(src + r0 * Ps + c0 + 4 * k);
          q[1][k] = *(const PDFMI_GLOBAL f32x4*)(src + r1 * Ps + c0 + 4 * k);
        }
#pragma unroll
      for (int c = 0; c < 12; ++c)
        if (c0 + c < P) {
          const int to = pos[c0 + c];
          if (to >= 0) {
            dst[r0 * kRow + to] = q[0][c >> 2][c & 3];
            dst[r1 * kRow + to] = q[1][c >> 2][c & 3];
          }
        }
    }
}

// Workgroup copy of rows x P elements from rows of stride Ps (global) into
// rows of stride P (LDS), eight loads in flight per thread; consecutive threads
// on consecutive elements, (row, column) advanced without a division.
template <int BS, typename T>
__device__ __forceinline__ void stage_rows(T* dst, const T* src, int rows, int P, int Ps) {
  const int ne = rows * P;
  const int drow = BS / P, dcol = BS - drow * P;
  int row = (int)threadIdx.x / P, col = (int)threadIdx.x - row * P;
  for (int e0 = threadIdx.x; e0 < ne; e0 += 8 * BS) {
    T r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      r[k] = ((const PDFMI_GLOBAL T*)src)[min(row, rows - 1) * Ps + col];  // clamped: every load in bounds
      row += drow;
      col += dcol;
      if (col >= P) {
        col -= P;
        ++row;
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = e0 + k * BS;
      if (e < ne) dst[e] = r[k];
    }
  }
}

// x*f for a set of flavours; see file header.  out is point-major [n][R].
// Each wave works on its own tiles of 64 points (fewer in small calls) with no workgroup barrier after
// the initial staging, so the knot searches and log transforms of some waves
// overlap the stencil gathers of others.  In-grid entries run a branch-free
// gather + FMA loop; the rare points outside the grid wait in the wave's list
// until they fill a pass.
constexpr int kWave = 64;

__device__ constexpr AlphasDev kNoAlphas{};

template <typename T>
__host__ __device__ constexpr size_t wave_record_bytes() {
  return (size_t)kWave * (sizeof(PointRec<T>) + 16 + 4);  // located points, then the points outside the grid
}
// Points outside the grid that a wave holds: 11 in FP64, 16 in FP32.
template <typename T>
constexpr int kSlowSlots = (int)(kWave * 20 / sizeof(SlowRec<T>));

// The outputs of the wave's ns points outside the grid, one lane per (point,
// requested column).  One point at a time across the wave left 64 - R lanes
// idle and paid each region's branch and a call with its weights in scratch
// memory: 1 % of the points outside cost 10^7 points of 13 columns 67 us (FP64
// with alpha_s, 711 -> 778) and 10 % 606; with the list 32 and 167.  col0:
// column 0 of grid row 0; colmap: stored column of each requested flavour, -1
// if absent (kCompact: rows in request order).
template <typename T, bool kGlobal, bool kCompact = false>
__device__ __forceinline__ void finish_slow(const SlowRec<T>* q, int ns, int R, const int* colmap, const T* col0,
                                            int Pp, double invL01, const LogEntry* lt, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int e = lane; e < ns * R; e += kWave) {
    const int k = e / R, j = e - k * R;
    const int c = colmap[j];
    T val = (T)0;
    if (c >= 0) val = rec_extrapolate<T, kGlobal>(q[k].r, q[k].mode, q[k].p0, q[k].p1, col0 + (kCompact ? j : c), Pp, invL01, lt);
    ((PDFMI_GLOBAL T*)q[k].out)[j] = val;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave's 64-point tile [pbeg, pbeg + tp): phase 1 (one lane per point,
// (xv, qv) = this lane's point) into the wave's LDS record, then the in-grid
// outputs, then the waiting points outside the grid (nslow of them before and
// after) if no further one has room in a pass.  obase = output row of point pbeg.
//
// Phase 2 walks the tile's outputs with consecutive lanes on consecutive
// output addresses: one lane per (point, flavour) for a flavour subset
// (G = 1), or per (point, group of G stored columns) when every stored column
// is requested in order (G * sizeof(T) = 16 bytes).  Reading the grid from
// global memory, groups start at min(G*j, R - G): the last group of a point
// overlaps the one before it and every store is full width (the shared
// column gets the same value twice).  Reading it from LDS, groups start at
// G*j (16-byte aligned LDS reads; rows are zero-padded to a multiple of G)
// and the last group stores only the columns below R.  kCompact: the LDS rows
// hold the request's columns in request order (0 for an absent flavour), so
// every request is walked in groups.
template <typename T, bool kLdsGrid, int G, bool kAlphas = false, bool kOverlap = !kLdsGrid, int kRowB = 0,
          bool kCompact = false>
__device__ __forceinline__ void wave_tile(const MemberDev& m, const Tables& tb, const int* scol, int R,
                                          const T* sgrid, const T* __restrict__ gvals, uint32_t gbytes,
                                          double xv, double qv, int tp, T* __restrict__ obase,
                                          unsigned long long* __restrict__ nerr, double invL01,
                                          unsigned char* rec, int& nslow, int lane, const AlphasDev& A,
                                          const AsView& av) {
  PointRec<T>* srec = reinterpret_cast<PointRec<T>*>(rec);            // [64]
  SlowRec<T>* sslow = reinterpret_cast<SlowRec<T>*>(srec + kWave);    // [kSlowSlots] points outside the grid
  const int Pp = kCompact ? kRowB / (int)sizeof(T) : (sizeof(T) == 8 ? m.P64 : m.P32);
  // bytes between consecutive Q^2 knots; a compile-time kRowB (the caller has
  // checked it) lets the four Q^2 rows of an LDS gather use immediate offsets
  const int rowb = kRowB ? kRowB : Pp * (int)sizeof(T);
  constexpr int kSlow = kLowX | kLowQ | kHighQ;
  // lane -> (point, flavour) or (point, column group) walk of the tile's outputs
  const int NE = G == 1 ? R : (R + G - 1) / G;
  const int e_p0 = lane / NE, e_j0 = lane - (lane / NE) * NE;
  const int e_dp = kWave / NE, e_dj = kWave - (kWave / NE) * NE;
  if constexpr (kAlphas) {  // alpha_s at the same points (fused evaluation), counted like pdf_alphas_q2
    const bool qbad = lane < tp && !(qv > 0.0 && qv < INFINITY);
    if (lane < tp) av.out[lane] = alphas_point(A, av, qv);
    const unsigned long long qb = __ballot(qbad);
    if (qb && lane == 0) atomicAdd(nerr, (unsigned long long)__popcll(qb));
  }
  bool bad = false, slow = false;
  PointRec<T> r;
  PointLoc L;
  if (lane < tp) {
    const QLoc<T> Q = locate_q<T>(m, tb, qv);
    L = locate_x<T>(m, tb, Q, xv, qv, r.w, r.v);
    bad = L.mode & kInvalid;
    slow = L.mode & kSlow;
    set_stencil(r, Q, L, rowb);
    srec[lane] = r;
  }
  const unsigned long long bal = __ballot(bad);
  if (bal && lane == 0) atomicAdd(nerr, (unsigned long long)__popcll(bal));
  // points outside the grid: into the wave's list, which is worked off after the tile's other outputs when
  // it has as many as one pass over the wave takes, and at the wave's end
  unsigned long long slow_mask = __ballot(slow);
  while (slow_mask) {
    if (nslow == kSlowSlots<T>) {
      finish_slow<T, !kLdsGrid, kCompact>(sslow, nslow, R, scol, kLdsGrid ? sgrid : gvals, Pp, invL01, tb.logt, lane);
      nslow = 0;
    }
    const int rank = __popcll(slow_mask & ((1ull << lane) - 1));
    const int take = min(kSlowSlots<T> - nslow, (int)__popcll(slow_mask));
    const bool mine = (slow_mask >> lane & 1) && rank < take;
    if (mine) {
      SlowRec<T>& d = sslow[nslow + rank];
      d.r = r;
      d.p0 = L.p0;
      d.p1 = L.p1;
      d.mode = L.mode;
      d.out = obase + lane * R;
    }
    slow_mask &= ~__ballot(mine);
    nslow += take;
  }
  // records written by this wave are read back by other lanes of the same wave
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  const __amdgpu_buffer_rsrc_t gr = buffer_rsrc(gvals, gbytes);
  const __amdgpu_buffer_rsrc_t orr = buffer_rsrc(obase, (uint32_t)(tp * R * (int)sizeof(T)));
  const int nev = tp * NE;
  int p = e_p0, j = e_j0;
  for (int e = lane; e < nev; e += kWave) {
    const PointRec<T>& pr = srec[p];
    const int po = pr.o;
    if (!(po & kRecSlow)) {
      T w[4], v[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        w[a] = pr.w[a];
        v[a] = pr.v[a];
      }
      const int s1 = pr.s1, sa = pr.sa, s3 = pr.s3;
      const bool inv = po & kRecInvalid;
      int c0;       // first output column of this entry
      int ccol;     // its stored column (-1: flavour absent from the grid)
      if constexpr (G == 1) {
        c0 = j;
        ccol = kCompact ? j : scol[j];
      } else {
        c0 = kOverlap ? min(G * j, R - G) : G * j;
        ccol = c0;
      }
      T res[G];
      if (inv) {
#pragma unroll
        for (int i = 0; i < G; ++i) res[i] = (T)NAN;
      } else if (G == 1 && ccol < 0) {
#pragma unroll
        for (int i = 0; i < G; ++i) res[i] = (T)0;
      } else {
        const int o0 = po + ccol * (int)sizeof(T);
        const int ox[4] = {o0, o0 + s1, o0 + s1 + sa, o0 + s1 + sa + s3};
        T F[G][4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const int oa = ox[a];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            T q[G];
            if constexpr (kLdsGrid) {
              const T* s = reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(sgrid) + oa + b * rowb);
              if constexpr (G > 1) {
                using V = typename VecOf<T, G>::type;  // 16-byte aligned: groups start at multiples of G
                const V vq = *reinterpret_cast<const V*>(s);
                __builtin_memcpy(q, &vq, sizeof(V));
              } else {
                q[0] = s[0];
              }
            } else {
              buf_load<T, G>(gr, oa, b * rowb, q);
            }
#pragma unroll
            for (int i = 0; i < G; ++i) F[i][a][b] = q[i];
          }
        }
#pragma unroll
        for (int i = 0; i < G; ++i) res[i] = interp_stencil<T>(F[i], w, v);
      }
      const int ob = (p * R + c0) * (int)sizeof(T);
      if (kOverlap || G * j + G <= R) {
        buf_store<T, G, kLdsGrid ? 0 : kStoreStream>(orr, ob, res);
      } else {
        // last group of a point without overlap: only the columns below R
#pragma unroll
        for (int i = 0; i < G - 1; ++i)
          if (i < R - G * j) buf_store<T, 1, kLdsGrid ? 0 : kStoreStream>(orr, ob + i * (int)sizeof(T), res + i);
      }
    }
    p += e_dp;
    j += e_dj;
    if (j >= NE) {
      j -= NE;
      ++p;
    }
  }
  if (nslow * R > kWave - R) {  // no room for another point in one pass
    finish_slow<T, !kLdsGrid, kCompact>(sslow, nslow, R, scol, kLdsGrid ? sgrid : gvals, Pp, invL01, tb.logt, lane);
    nslow = 0;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

#ifndef PDFMI_WAVES_PER_EU
#define PDFMI_WAVES_PER_EU 1
#endif

// Bytes of the alpha_s block a kernel stages: all of it, or without its
// logarithm table when the member's (equal) one is in LDS already.
__host__ __device__ static inline int alphas_staged_bytes(const AlphasDev& A, bool member_tables) {
  return member_tables ? A.logt_off : A.bytes;
}

// LDS bytes of a staged grid, up to the 16-byte aligned table behind it.
template <typename T>
__host__ __device__ constexpr size_t grid_lds_bytes(int elems) {
  return ((size_t)elems * sizeof(T) + 15) & ~(size_t)15;
}

// LDS layout of k_xfxq2 and k_batched: [location tables][column map][per-wave
// records][grid values], the tables only when they are staged (kLdsTables)
// and the grid only when it is staged (kLdsGrid, which implies kLdsTables).
template <typename T, bool kLdsGrid, int G, int BS, bool kLdsTables, bool kAlphas>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(kAlphas ? 4 : PDFMI_WAVES_PER_EU)))
void k_xfxq2(MemberDev m, ReqCols rc, const double* __restrict__ X, const double* __restrict__ Q2, int64_t n,
             T* __restrict__ out, unsigned long long* __restrict__ nerr, int lds_grid_elems, double invL01,
             AlphasDev A, double* __restrict__ aout, int tile_pts) {
  static_assert(kLdsTables || !kLdsGrid, "a staged grid needs staged tables");
  constexpr int kWaves = BS / kWave;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* stbl = smem;
  int* scol = reinterpret_cast<int*>(smem + (kLdsTables ? m.tbl_bytes : 0));
  unsigned char* srec = reinterpret_cast<unsigned char*>(scol + kMaxReq);
  T* sgrid = reinterpret_cast<T*>(srec + kWaves * wave_record_bytes<T>());
  // alpha_s table (fused alpha_s output only), after the staged grid, 16-byte aligned
  unsigned char* sas = reinterpret_cast<unsigned char*>(sgrid) + (kLdsGrid ? grid_lds_bytes<T>(lds_grid_elems) : 0);
  AsView av{sas, nullptr, nullptr};
  if constexpr (kAlphas) stage_copy<BS>(sas, A.tables, alphas_staged_bytes(A, kLdsTables));
  if constexpr (kLdsTables) stage_copy<BS>(stbl, m.tables, m.tbl_bytes);
  for (int i = threadIdx.x; i < rc.n; i += BS) scol[i] = rc.col[i];
  const T* __restrict__ gvals = member_values<T>(m);
  const uint32_t gbytes = (uint32_t)((sizeof(T) == 8 ? m.elems64 : m.elems32) * (int64_t)sizeof(T));
  if constexpr (kLdsGrid) stage_copy<BS>(sgrid, gvals, (int64_t)lds_grid_elems * (int64_t)sizeof(T));
  __syncthreads();
  const Tables tb = tables_at(kLdsTables ? stbl : m.tables, m);
  av.logt = kLdsTables ? tb.logt : reinterpret_cast<const LogEntry*>(sas + A.logt_off);

  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  unsigned char* rec = srec + wv * wave_record_bytes<T>();
  const int R = rc.n;
  const int pts = kLdsTables ? kWave : tile_pts;  // points of a tile, at most kWave
  const int64_t ntiles = (n + pts - 1) / pts;
  const int64_t stride = (int64_t)gridDim.x * kWaves;
  int64_t tile = (int64_t)blockIdx.x * kWaves + wv;
  // the next tile's (x, Q^2) are loaded before the current tile is processed
  double xc = 0.0, qc = 0.0;
  int nslow = 0;  // points outside the grid that wait (uniform over the wave)
  if (tile < ntiles && tile * pts + lane < n) {
    xc = X[tile * pts + lane];
    qc = Q2[tile * pts + lane];
  }
  for (; tile < ntiles; tile += stride) {
    const int64_t pbeg = tile * pts;
    const int tp = (int)min((int64_t)pts, n - pbeg);
    const int64_t nxt = pbeg + stride * pts + lane;
    double xn = 0.0, qn = 0.0;
    if (nxt < n) {
      xn = X[nxt];
      qn = Q2[nxt];
    }
    if constexpr (kAlphas) av.out = aout + pbeg;
    wave_tile<T, kLdsGrid, G, kAlphas>(m, tb, scol, R, sgrid, gvals, gbytes, xc, qc, tp, out + pbeg * R, nerr, invL01, rec,
                                       nslow, lane, A, av);
    xc = xn;
    qc = qn;
  }
  if (nslow > 0)
    finish_slow<T, !kLdsGrid>(reinterpret_cast<const SlowRec<T>*>(rec + kWave * sizeof(PointRec<T>)), nslow, R, scol,
                            kLdsGrid ? sgrid : gvals, sizeof(T) == 8 ? m.P64 : m.P32, invL01, tb.logt, lane);
}

// Location only (sub-grid, cells, region), one lane per point.
__global__ __launch_bounds__(256) void k_locate(MemberDev m, const double* __restrict__ X,
                                                const double* __restrict__ Q2, int64_t n,
                                                int32_t* __restrict__ ko, int32_t* __restrict__ ixo,
                                                int32_t* __restrict__ iqo, int8_t* __restrict__ rego) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double w[4], v[4];
    const Tables tb = tables_at(m.tables, m);
    const QLoc<double> Q = locate_q<double>(m, tb, Q2[i]);
    const PointLoc L = locate_x<double>(m, tb, Q, X[i], Q2[i], w, v);
    const bool bad = L.mode & kInvalid;
    ko[i] = bad ? -1 : Q.kiq >> 16;
    ixo[i] = bad ? -1 : L.ix;
    iqo[i] = bad ? -1 : Q.kiq & 0xffff;
    rego[i] = (int8_t)(L.mode & (kLowX | kLowQ | kHighQ | kInvalid));
  }
}

// alpha_s(Q^2) at n points (paper section 2.3): segment (repeated knot =
// threshold, the upper segment owns it), FP64 knot search, cubic Hermite in
// ln Q^2 with one-sided slopes at segment ends, constant outside the knots.
// The table block (at most 28 KB) is staged in LDS once per workgroup; four
// independent evaluations in flight per lane.  Vector work (61 % busy) and the
// 16 bytes per point bound it: 10^7 points 86.5 us with the library's logarithm
// and per-segment searches, 37 now; moving the bytes alone takes 31.
__global__ __launch_bounds__(256) void k_alphas(AlphasDev A, const double* __restrict__ Q2, int64_t n,
                                                double* __restrict__ out, unsigned long long* __restrict__ nerr) {
  extern __shared__ __align__(16) unsigned char sas[];
  stage_copy<256>(sas, A.tables, A.bytes);
  const AsView av{sas, reinterpret_cast<const LogEntry*>(sas + A.logt_off), nullptr};
  __syncthreads();
  // each wave takes 256 consecutive points per step, lane l the points l + 64 j
  // (j = 0..3): every load and store instruction covers 512 contiguous bytes.
  // The next step's Q^2 are loaded before the current step is evaluated.
  const int lane = threadIdx.x & 63;
  const int64_t nchunks = (n + 255) / 256;
  const int64_t wstride = (int64_t)gridDim.x * (256 / 64);
  int64_t c = (int64_t)blockIdx.x * (256 / 64) + (threadIdx.x >> 6);
  double q[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t i = c * 256 + j * 64 + lane;
    q[j] = i < n ? Q2[i] : 1.0;
  }
  unsigned long long cnt = 0;
  for (; c < nchunks; c += wstride) {
    double qn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = (c + wstride) * 256 + j * 64 + lane;
      qn[j] = i < n ? Q2[i] : 1.0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = c * 256 + j * 64 + lane;
      const double r = alphas_point(A, av, q[j]);
      if (i < n) out[i] = r;
      cnt += __popcll(__ballot(i < n && !(q[j] > 0.0 && q[j] < INFINITY)));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = qn[j];
  }
  if (cnt && lane == 0) atomicAdd(nerr, cnt);
}

// ---------------------------------------------------------------------------------------
// Launchers (host side, called by pdfmi.cpp)

// Location tables up to this size are staged in LDS (typical sets need
// 10-40 KB: a few hundred knots of 8 bytes, 48 bytes per x cell, 80 per Q^2
// cell, the hints and 2 KB for the logarithm); larger ones are read from
// global memory.
constexpr size_t kMaxLdsTables = 64 * 1024;
static bool tables_fit(const MemberDev& m) { return (size_t)m.tbl_bytes <= kMaxLdsTables; }

// LDS bytes of the alpha_s table staged for a fused alpha_s output (member_tables: beside the member's tables).
size_t alphas_lds_bytes(const AlphasDev* A, bool member_tables) {
  return A ? (size_t)alphas_staged_bytes(*A, member_tables) : 0;
}

// LDS bytes of k_xfxq2 other than the staged grid, for a block of bs threads.
static size_t shared_bytes(const MemberDev& m, bool f32, int bs, bool tables) {
  return (tables ? (size_t)m.tbl_bytes : 0) + kMaxReq * 4 +
         (bs / kWave) * (f32 ? wave_record_bytes<float>() : wave_record_bytes<double>());
}
constexpr int kBlockGlobal = 256;   // tables and grid read from global memory
// Small calls read the tables in place (staging tens of KB costs a workgroup
// more than the few entries its points need) and are bound by latency: the
// kernel arguments, the table reads of the location and then one gather round
// after another.  Their tiles are halved until the call has kSmallWaves waves
// per compute unit, down to the 8 points whose column groups fill about one
// round.  A call that has that many full tiles stages the tables.  Measured on
// 256 compute units, FP64, 11 and 13 columns (64-point tiles, staged from
// 32768 points on, then this rule): 10^3 points 8.2 -> 5.7 and 11.7 -> 7.9 us,
// 10^4 8.5 -> 5.8 and 15.4 -> 9.1, 65000 11.1 -> 8.7 and 20.0 -> 13.9; at 10^5
// staged full tiles take 11.2 and 19.2, in place 11.7 and 19.2, staged tiles
// of 32 points 11.7 and 19.0.  8 or 16 waves per compute unit: 32000 points
// 7.5 against 6.9 us.
constexpr int kSmallWaves = 4;
constexpr int kMinTilePts = 8;
constexpr int kBlockTables = 512;   // tables staged in LDS, grid read from global memory
constexpr int kBlockLds = 1024;     // tables and grid staged once per workgroup in LDS
constexpr int kBlockLdsSmall = 768; // the same, where only fewer waves' records fit beside them
size_t xfxq2_shared_bytes(const MemberDev& m, bool f32, bool small) {
  return shared_bytes(m, f32, small ? kBlockLdsSmall : kBlockLds, true);
}

// Launch context: the alpha_s table and output of a fused evaluation (A and
// aout null when alpha_s is not requested).
struct AsOut {
  const AlphasDev* A;
  double* aout;
};

template <typename T, int G, int BS, bool kLdsGrid, bool kLdsTables, bool kAlphas>
static hipError_t launch_one(const MemberDev& m, const ReqCols& rc, const double* x, const double* q2, int64_t n,
                             T* out, unsigned long long* nerr, int lds_grid_elems, double invL01, int64_t nb,
                             size_t shm, const AsOut& ao, hipStream_t s, int tile_pts = kWave) {
  const void* fn = reinterpret_cast<const void*>(&k_xfxq2<T, kLdsGrid, G, BS, kLdsTables, kAlphas>);
  hipError_t e = allow_dynamic_lds(fn, shm);
  if (e != hipSuccess) return e;
  const AlphasDev A = ao.A ? *ao.A : AlphasDev{};
  hipLaunchKernelGGL((k_xfxq2<T, kLdsGrid, G, BS, kLdsTables, kAlphas>), dim3((unsigned)nb), dim3(BS), shm, s, m, rc, x, q2,
                     n, out, nerr, lds_grid_elems, invL01, A, ao.aout, tile_pts);
  return hipGetLastError();
}

template <typename T, int G, bool kAlphas>
static hipError_t launch_xfxq2_g(const MemberDev& m, const ReqCols& rc, const double* x, const double* q2,
                                 int64_t n, T* out, unsigned long long* nerr, int lds_grid_elems,
                                 double invL01, const LaunchCfg& cfg, const AsOut& ao, hipStream_t s) {
  const int n_cu = cfg.n_cu;
  const bool f32 = sizeof(T) == 4;
  const size_t as_bytes = alphas_lds_bytes(ao.A, true);
  if (lds_grid_elems > 0) {
    const size_t values = grid_lds_bytes<T>(lds_grid_elems) + as_bytes;
    const bool large = shared_bytes(m, f32, kBlockLds, true) + values <= 160 * 1024;
    const size_t shm = shared_bytes(m, f32, large ? kBlockLds : kBlockLdsSmall, true) + values;
    const int per_cu = max(1, (int)(160 * 1024 / shm));
    const int64_t ntiles = (n + kBlockLds - 1) / kBlockLds;
    const int64_t nb = min(ntiles, (int64_t)n_cu * per_cu);
    if (!large)
      return launch_one<T, G, kBlockLdsSmall, true, true, kAlphas>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, nb,
                                                                   shm, ao, s);
    return launch_one<T, G, kBlockLds, true, true, kAlphas>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, nb, shm, ao,
                                                   s);
  }
  const int64_t full = (int64_t)n_cu * kSmallWaves * kWave;  // points that give every small wave a full tile
  if (tables_fit(m) && n >= full) {
    const size_t shm = shared_bytes(m, f32, kBlockTables, true) + as_bytes;
    // two workgroups are resident per compute unit; more than that are
    // launched only while every wave still has about three tiles of its own,
    // so that the staging of the tables is paid once for several tiles (FP32,
    // 1.2e6 points: 72 us with one tile per wave, 63 with five) and long
    // launches keep a queue that evens out the end (FP64, 1e7 points: 760 us
    // with two workgroups per compute unit, 726 with 16 or more)
    const int64_t ntiles = (n + kBlockTables - 1) / kBlockTables;
    const int64_t per_cu = ntiles / (3 * (int64_t)n_cu);
    const int64_t nb =
        min(ntiles, (int64_t)n_cu * min((int64_t)cfg.blocks_per_cu, max((int64_t)2, per_cu & ~(int64_t)1)));
    return launch_one<T, G, kBlockTables, false, true, kAlphas>(m, rc, x, q2, n, out, nerr, 0, invL01, nb, shm, ao, s);
  }
  const size_t shm = shared_bytes(m, f32, kBlockGlobal, false) + alphas_lds_bytes(ao.A, false);
  int tile_pts = kWave;
  for (int64_t f = full; tile_pts > kMinTilePts && n < f; f /= 2) tile_pts /= 2;
  const int block_pts = kBlockGlobal / kWave * tile_pts;
  const int64_t ntiles = (n + block_pts - 1) / block_pts;
  const int64_t nb = min(ntiles, (int64_t)n_cu * cfg.blocks_per_cu);
  return launch_one<T, G, kBlockGlobal, false, false, kAlphas>(m, rc, x, q2, n, out, nerr, 0, invL01, nb, shm, ao, s,
                                                               tile_pts);
}

// The vectorised kernel serves requests for every stored column in load order.
// Its groups of G columns need at least G of them.
static bool all_columns(const MemberDev& m, const ReqCols& rc, int G) {
  if (rc.n != m.P || rc.n < G) return false;
  for (int j = 0; j < rc.n; ++j)
    if (rc.col[j] != j) return false;
  return true;
}

// Copy of the requested columns of `rows` grid rows (stride Ps) in request
// order, rows of Rp values; absent flavours and padding are 0.
template <typename T>
__device__ __forceinline__ void compact_one(const T* src, int64_t e, int Ps, const ReqCols& rc, int Rp, T* dst) {
  const int64_t row = e / Rp;
  const int j = (int)(e - row * Rp);
  const int c = j < rc.n ? rc.col[j] : -1;
  dst[e] = c >= 0 ? src[row * Ps + c] : (T)0;
}
template <typename T>
__global__ void k_compact(const T* __restrict__ src, int64_t elems, int Ps, ReqCols rc, int Rp, T* __restrict__ dst) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < elems) compact_one(src, e, Ps, rc, Rp, dst);
}
// All copies of a plan in one launch (100 copies of 5 of 11 columns added 390 us
// to the making of a plan with a launch each; 75 now, their allocation included).
__global__ void k_compact_jobs(const CompactJob* __restrict__ jobs, int n) {
  for (int i = blockIdx.y; i < n; i += gridDim.y) {
    const CompactJob& job = jobs[i];
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < job.elems; e += (int64_t)gridDim.x * blockDim.x)
      compact_one(job.src, e, job.Ps, job.rc, job.Rp, job.dst);
  }
}
hipError_t launch_compact_jobs(const CompactJob* jobs, int n, int64_t max_elems, hipStream_t s) {
  const dim3 grid((unsigned)min((max_elems + 255) / 256, (int64_t)64), (unsigned)min(n, 4096));
  hipLaunchKernelGGL(k_compact_jobs, grid, dim3(256), 0, s, jobs, n);
  return hipGetLastError();
}

hipError_t launch_compact(const MemberDev& m, const ReqCols& rc, bool f32, int Rp, void* dst, hipStream_t s) {
  const int64_t elems = (int64_t)m.rows * Rp;
  const dim3 nb((unsigned)((elems + 255) / 256));
  if (f32)
    hipLaunchKernelGGL(k_compact<float>, nb, dim3(256), 0, s, m.v32, elems, m.P32, rc, Rp, static_cast<float*>(dst));
  else
    hipLaunchKernelGGL(k_compact<double>, nb, dim3(256), 0, s, m.v64, elems, m.P64, rc, Rp,
                       static_cast<double*>(dst));
  return hipGetLastError();
}

// A, aout: the alpha_s table and output of a fused evaluation, or null.
// compact: the member's values are a copy compacted to the request (rc.col[j]
// is j, or -1 for an absent flavour): walked in groups like a request for all
// columns.
hipError_t launch_xfxq2_f64(const MemberDev& m, const ReqCols& rc, const double* x, const double* q2, int64_t n,
                            double* out, unsigned long long* nerr, int lds_grid_elems, double invL01,
                            const LaunchCfg& cfg, const AlphasDev* A, double* aout, bool compact, hipStream_t s) {
  const AsOut ao{aout ? A : nullptr, aout};
  const bool vec = cfg.vector_cols && (compact ? layout_group(rc.n, false) == 2 : all_columns(m, rc, 2));
  if (aout)
    return vec ? launch_xfxq2_g<double, 2, true>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s)
               : launch_xfxq2_g<double, 1, true>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s);
  return vec ? launch_xfxq2_g<double, 2, false>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s)
             : launch_xfxq2_g<double, 1, false>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s);
}

hipError_t launch_xfxq2_f32(const MemberDev& m, const ReqCols& rc, const double* x, const double* q2, int64_t n,
                            float* out, unsigned long long* nerr, int lds_grid_elems, double invL01,
                            const LaunchCfg& cfg, const AlphasDev* A, double* aout, bool compact, hipStream_t s) {
  const AsOut ao{aout ? A : nullptr, aout};
  const bool vec = cfg.vector_cols && (compact ? layout_group(rc.n, true) == 4 : all_columns(m, rc, 4));
  if (!vec && compact && layout_group(rc.n, true) == 2)
    return aout ? launch_xfxq2_g<float, 2, true>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s)
                : launch_xfxq2_g<float, 2, false>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s);
  if (aout)
    return vec ? launch_xfxq2_g<float, 4, true>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s)
               : launch_xfxq2_g<float, 1, true>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s);
  return vec ? launch_xfxq2_g<float, 4, false>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s)
             : launch_xfxq2_g<float, 1, false>(m, rc, x, q2, n, out, nerr, lds_grid_elems, invL01, cfg, ao, s);
}

hipError_t launch_locate(const MemberDev& m, const double* x, const double* q2, int64_t n, int32_t* k, int32_t* ix,
                         int32_t* iq, int8_t* reg, int n_cu, hipStream_t s) {
  const int64_t nb = min((n + 255) / 256, (int64_t)n_cu * 16);
  hipLaunchKernelGGL(k_locate, dim3((unsigned)nb), dim3(256), 0, s, m, x, q2, n, k, ix, iq, reg);
  return hipGetLastError();
}

hipError_t launch_alphas(const AlphasDev& A, const double* q2, int64_t n, double* out, unsigned long long* nerr,
                         int n_cu, hipStream_t s) {
  const int64_t nb = min((n + 1023) / 1024, (int64_t)n_cu * 8);
  hipLaunchKernelGGL(k_alphas, dim3((unsigned)nb), dim3(256), (size_t)A.bytes, s, A, q2, n, out, nerr);
  return hipGetLastError();
}

}  // namespace pdfmi

namespace pdfmi {

// ---------------------------------------------------------------------------------------
// Monte-Carlo luminosity chunk sum (the integrand-shaped load of the paper's
// section 4.1): S = sum_i alpha_s(Q^2_i) * sum_j xf1[i][j] * xf2[i][j], FP64,
// in a fixed order that depends only on n: stage 1 gives one partial per
// block of kMcBlock points (each thread sums its strided points in index
// order, then a fixed binary tree in LDS); stage 2 sums the partials with the
// same tree in one workgroup.  Bit-identical across runs.
constexpr int kMcThreads = 256;
constexpr int kMcBlock = 1024;  // 4 points per thread: a 1e6-point chunk spans ~1000 blocks

// Sum of 256 values in the order of a binary tree (t + 128, t + 64, ..., t + 1),
// given values t, t + 64, t + 128, t + 192 in lane t of one wave: the first two
// levels within the lane, the others across lanes.
__device__ __forceinline__ double wave_tree_sum(double v0, double v1, double v2, double v3) {
  double v = (v0 + v2) + (v1 + v3);
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s);
  return v;  // in lane 0
}

// The same over a workgroup's 256 values, one barrier; the sum in thread 0.
__device__ __forceinline__ double block_tree_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  const int t = threadIdx.x & 63;
  return threadIdx.x < 64 ? wave_tree_sum(sh[t], sh[t + 64], sh[t + 128], sh[t + 192]) : 0.0;
}

// Stage 1 when the rows do not fit LDS (many flavours): the same order read
// straight from global memory.
template <typename T>
__global__ __launch_bounds__(kMcThreads) void k_mc_partial_direct(const T* __restrict__ xf1,
                                                                  const T* __restrict__ xf2, int P,
                                                                  const double* __restrict__ as, int64_t n,
                                                                  double* __restrict__ partial) {
  __shared__ double sh[kMcThreads];
  const int64_t beg = (int64_t)blockIdx.x * kMcBlock;
  const int64_t end = min(beg + kMcBlock, n);
  double acc = 0.0;
  for (int k = 0; k < kMcBlock / kMcThreads; ++k) {
    const int64_t i = beg + threadIdx.x + (int64_t)kMcThreads * k;
    if (i < end) {
      double lum = 0.0;
      for (int j = 0; j < P; ++j) lum = fma((double)xf1[i * P + j], (double)xf2[i * P + j], lum);
      acc = fma(as[i], lum, acc);
    }
  }
  const double s = block_tree_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Stage 1.  The block's points are taken 256 at a time: their xf1 and xf2
// rows (contiguous in memory) are copied to LDS with coalesced loads, then
// thread t forms sum_j xf1 xf2 of its point in flavour order and accumulates
// alpha_s times it -- thread t sees points beg + t + 256 k in increasing k.
template <typename T>
__global__ __launch_bounds__(kMcThreads) void k_mc_partial(const T* __restrict__ xf1, const T* __restrict__ xf2,
                                                           int P, const double* __restrict__ as, int64_t n,
                                                           double* __restrict__ partial) {
  __shared__ double sh[kMcThreads];
  extern __shared__ __align__(16) unsigned char mc_smem[];
  T* s1 = reinterpret_cast<T*>(mc_smem);  // [256][P]
  T* s2 = s1 + kMcThreads * P;            // [256][P]
  const int64_t beg = (int64_t)blockIdx.x * kMcBlock;
  const int64_t end = min(beg + kMcBlock, n);
  double acc = 0.0;
  for (int k = 0; k < kMcBlock / kMcThreads; ++k) {
    const int64_t p0 = beg + (int64_t)kMcThreads * k;
    if (p0 >= end) break;  // uniform across the block
    const int np = (int)min((int64_t)kMcThreads, end - p0);
    __syncthreads();       // previous step's rows consumed
    for (int e = threadIdx.x; e < np * P; e += kMcThreads) {
      s1[e] = xf1[p0 * P + e];
      s2[e] = xf2[p0 * P + e];
    }
    __syncthreads();
    if ((int)threadIdx.x < np) {
      double lum = 0.0;
      for (int j = 0; j < P; ++j) lum = fma((double)s1[threadIdx.x * P + j], (double)s2[threadIdx.x * P + j], lum);
      acc = fma(as[p0 + threadIdx.x], lum, acc);
    }
  }
  const double s = block_tree_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ __launch_bounds__(kMcThreads) void k_mc_final(const double* __restrict__ partial, int64_t np,
                                                         double* __restrict__ sum_out) {
  __shared__ double sh[kMcThreads];
  double acc = 0.0;
  for (int64_t i0 = threadIdx.x; i0 < np; i0 += 8 * kMcThreads) {  // eight loads in flight, added in order
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = partial[min(i0 + k * kMcThreads, np - 1)];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i0 + k * kMcThreads < np) acc += v[k];
  }
  const double s = block_tree_sum(acc, sh);
  if (threadIdx.x == 0) *sum_out = s;
}

int64_t mc_partials(int64_t n) { return (n + kMcBlock - 1) / kMcBlock; }

template <typename T>
hipError_t launch_mc_sum(const T* xf1, const T* xf2, int P, const double* as, int64_t n, double* partial,
                         double* sum_out, hipStream_t s) {
  const int64_t np = mc_partials(n);
  if (np > 0) {
    const size_t shm = (size_t)2 * kMcThreads * P * sizeof(T);
    if (shm <= 96 * 1024) {
      hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&k_mc_partial<T>), shm);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(k_mc_partial<T>, dim3((unsigned)np), dim3(kMcThreads), shm, s, xf1, xf2, P, as, n, partial);
    } else {
      hipLaunchKernelGGL(k_mc_partial_direct<T>, dim3((unsigned)np), dim3(kMcThreads), 0, s, xf1, xf2, P, as, n,
                         partial);
    }
  }
  hipLaunchKernelGGL(k_mc_final, dim3(1), dim3(kMcThreads), 0, s, partial, np, sum_out);
  return hipGetLastError();
}
// Fused Monte-Carlo chunk sum: the same S as xfxq2(x1) + xfxq2(x2) +
// alpha_s + the chunk sum above, without writing the PDF values out (24 bytes
// of input per point instead of 24 + 2 R sizeof(T) out and back in).  Each
// 256-thread quarter of a workgroup takes one kMcBlock-point block of the
// chunk, each thread its points beg + t + 256 k in increasing k: one lane per
// point locates x1 and x2, evaluates every requested flavour of both with the
// same device functions as k_xfxq2, forms sum_j xf1_j xf2_j in flavour order
// and accumulates alpha_s times it -- the summation order of k_mc_partial, so
// both paths give bit-identical sums.  The grid is staged in LDS when it
// fits (kLdsGrid), if need be with the tables left in place (kStaged): they are
// read a few times a point and mostly from the vector cache, the grid 32 times
// a flavour (10^6 points, FP64, 11 columns of 50 x 33 knots: grid and tables in
// global memory 1226 us, grid in LDS 95; at 50 x 32 all in LDS 101).  In FP32
// the LDS rows are padded with zeros to a multiple of kGW = 4 columns when that
// fits too, and the stencils are then read four columns at a time, as from
// global memory: one 16-byte read
// brings four columns of a stencil row (a random-row LDS gather of 16-byte reads
// delivers 2.3x the values per clock of 4-byte reads; from global memory 10^6
// points of 13 columns take 464 us, column by column 1185).  The flavour loop then
// walks a list of column-group steps built once per workgroup from the
// request: a step reads one group and applies the terms of the next 1..kGW
// requested flavours whose columns fall in it, in request order, so the sum
// is still formed flavour by flavour in that order; a flavour absent from the
// grid is a step of its own with no read.  Otherwise the rows keep stride P
// and each requested column is read on its own (kGW = 1), as in FP64: pairs
// of FP64 columns measured no faster than single 8-byte reads (with rows of
// 12 columns every stencil row starts on a 32-byte boundary and the reads of
// one instruction use half of the banks; padding the x stride by 16 bytes
// against that brought the pairs level with single reads, not below).
constexpr int kMcFusedBS = 4 * kMcThreads;
constexpr int kStepAbsent = -1;   // a step whose flavour is absent from the grid
constexpr int kStepOrdered = 1 << 19;  // the step's terms are the group's columns 0, 1, ... in order

// Column-group steps of a request (see above) into st[1..], their count into st[0].
// Step: group's first column (bits 0-15), term count (16-18), kStepOrdered,
// and the column within the group of term t in bits 20 + 2t, 21 + 2t.
template <int kGW>
__device__ __forceinline__ void mc_build_steps(const ReqCols& rc, int* st) {
  int ns = 0;
  for (int j = 0; j < rc.n;) {
    const int c = rc.col[j];
    if (c < 0) {
      st[1 + ns++] = kStepAbsent;
      ++j;
      continue;
    }
    const int g0 = c & ~(kGW - 1);
    int nt = 1, sel = c - g0;
    bool ordered = c == g0;
    while (nt < kGW && j + nt < rc.n && rc.col[j + nt] >= 0 && (rc.col[j + nt] & ~(kGW - 1)) == g0) {
      sel |= (rc.col[j + nt] - g0) << (2 * nt);
      ordered = ordered && rc.col[j + nt] - g0 == nt;
      ++nt;
    }
    st[1 + ns++] = g0 | (nt << 16) | (ordered ? kStepOrdered : 0) | (sel << 20);
    j += nt;
  }
  st[0] = ns;
}

// Element e (uniform) of a kGW-array of values held in registers.
template <typename T, int kGW>
__device__ __forceinline__ T mc_pick(const T (&f)[kGW], int e) {
  if constexpr (kGW == 1) {
    return f[0];
  } else if constexpr (kGW == 2) {
    return e ? f[1] : f[0];
  } else {
    static_assert(kGW == 4, "column groups of 2 or 4");
    return e == 0 ? f[0] : (e == 1 ? f[1] : (e == 2 ? f[2] : f[3]));
  }
}

// A located point's stencil in the values read by k_mc_fused (row stride P):
// element offset of each x knot's first row.
struct McOrigin {
  int x[4];
};
__device__ __forceinline__ McOrigin mc_origin(const PointLoc& L, int nqp, int P) {
  McOrigin o;
  o.x[0] = (int)__umul24((unsigned)L.row, (unsigned)P);
  const int sa = (int)__umul24((unsigned)nqp, (unsigned)P);
  o.x[1] = o.x[0] + (L.s1 ? sa : 0);
  o.x[2] = o.x[1] + sa;
  o.x[3] = o.x[2] + (L.s3 ? sa : 0);
  return o;
}

// One flavour of one located point, the value k_xfxq2 writes for it: NaN for
// an invalid point, 0 for a flavour absent from the grid, the stencil sum
// inside the grid, the extrapolation formula outside.  g points at the
// flavour's column of grid row 0; P is the row stride of the values read.
template <typename T, bool kMaySlow>
__device__ __forceinline__ T mc_value(const T* g, const PointLoc& L, const McOrigin& o, const T w[4], const T v[4],
                                      int P, int col, double invL01, const LogEntry* lt) {
  if (L.mode & kInvalid) return (T)NAN;
  if (col < 0) return (T)0;
  if (!kMaySlow || !(L.mode & (kLowX | kLowQ | kHighQ))) {
    T F[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) F[a][b] = g[o.x[a] + b * P];
    return interp_stencil<T>(F, w, v);
  }
  return (T)extrap_entry<T, false>(g + o.x[0], o.x[1] - o.x[0], o.x[2] - o.x[1], o.x[3] - o.x[2], P, L.mode, w[0], w[1],
                                   w[2], w[3], v[0], v[1], v[2], v[3], L.p0, L.p1, invL01, lt);
}

// What k_mc_fused stages of the tables: the logarithm's alone (an extrapolated
// value waits for up to four logarithms, one after another), alpha_s with it,
// or the member's location tables too.
enum McTables { kMcInPlace, kMcAlphas, kMcAll };

__host__ __device__ static inline int mc_alphas_bytes(const AlphasDev& A, McTables staged) {
  return staged == kMcInPlace ? A.bytes - A.logt_off : alphas_staged_bytes(A, staged == kMcAll);
}

template <typename T, bool kLdsGrid, int kGW, McTables kStaged = kMcAll>
__global__ __launch_bounds__(kMcFusedBS) void k_mc_fused(MemberDev m, ReqCols rc, AlphasDev A,
                                                         const double* __restrict__ X1,
                                                         const double* __restrict__ X2,
                                                         const double* __restrict__ Q2, int64_t n,
                                                         double* __restrict__ partial,
                                                         unsigned long long* __restrict__ nerr, double invL01,
                                                         int split) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr bool kLdsTables = kStaged == kMcAll;
  unsigned char* stbl = smem;
  unsigned char* sas = smem + (kLdsTables ? m.tbl_bytes : 0);
  const int as_bytes = mc_alphas_bytes(A, kStaged);
  double* tree = reinterpret_cast<double*>(sas + as_bytes);  // [4][256], twice when split
  int* scol = reinterpret_cast<int*>(tree + (split ? 2 : 1) * kMcFusedBS);  // [kMaxReq]
  int* sstep = scol + kMaxReq;                            // [kMaxReq + 4] column-group steps (kGW > 1)
  T* sgrid = reinterpret_cast<T*>(sstep + kMaxReq + 4);   // 16-byte aligned: 2 kMaxReq + 4 ints

  if constexpr (kLdsTables) stage_copy<kMcFusedBS>(stbl, m.tables, m.tbl_bytes);
  stage_copy<kMcFusedBS>(sas, A.tables + (kStaged == kMcInPlace ? A.logt_off : 0), as_bytes);
  for (int i = threadIdx.x; i < rc.n; i += kMcFusedBS) scol[i] = rc.col[i];
  const int Pp = sizeof(T) == 8 ? m.P64 : m.P32;
  const T* __restrict__ gvals = member_values<T>(m);
  // row stride of the values read below: in LDS P, or P rounded up to whole
  // column groups (<= Pp, whose padding columns are zero in global memory)
  const int P = kLdsGrid ? (m.P + kGW - 1) & ~(kGW - 1) : Pp;
  if constexpr (kGW > 1)
    if (threadIdx.x == 0) mc_build_steps<kGW>(rc, sstep);
  if constexpr (kLdsGrid) stage_rows<kMcFusedBS>(sgrid, gvals, m.rows, P, Pp);
  __syncthreads();
  Tables tb = tables_at(kLdsTables ? stbl : m.tables, m);
  if constexpr (!kLdsTables) tb.logt = reinterpret_cast<const LogEntry*>(sas + (kStaged == kMcAlphas ? A.logt_off : 0));
  const AsView av{kStaged == kMcInPlace ? A.tables : sas, tb.logt, nullptr};
  const T* grid = kLdsGrid ? sgrid : gvals;

  const int q = threadIdx.x / kMcThreads, t = threadIdx.x % kMcThreads;
  const int R = rc.n;
  const int64_t nmb = (n + kMcBlock - 1) / kMcBlock;
  const int per_wg = split ? 1 : 4;  // blocks of points a workgroup has in hand
  for (int64_t mb0 = (int64_t)blockIdx.x * per_wg; mb0 < nmb; mb0 += (int64_t)gridDim.x * per_wg) {
    const int64_t mb = split ? mb0 : mb0 + q;
    const int64_t beg = mb * kMcBlock, end = min(beg + (int64_t)kMcBlock, n);
    double acc = 0.0, as1 = 0.0;
    for (int k = split ? q : 0; k < (split ? q + 1 : kMcBlock / kMcThreads); ++k) {
      const int64_t i = beg + t + (int64_t)kMcThreads * k;
      const bool live = mb < nmb && i < end;
      double x1 = 0.5, x2 = 0.5, q2 = 10.0;
      if (live) {
        x1 = X1[i];
        x2 = X2[i];
        q2 = Q2[i];
      }
      // Q^2 weights: a valid point inside the grid in Q^2 has Qs.v (an invalid
      // one's value is NaN, an extrapolated one's Q^2 weights are unused
      // unless Q^2 is inside), so both lookups read them from Qs
      T w1[4], w2[4], vx[4];
      const QLoc<T> Qs = locate_q<T>(m, tb, q2);  // shared Q^2: located once for both lookups
      const PointLoc L1 = locate_x<T>(m, tb, Qs, x1, q2, w1, vx);
      const PointLoc L2 = locate_x<T>(m, tb, Qs, x2, q2, w2, vx);
      const T* v = Qs.v;
      const double as = alphas_point(A, av, q2);
      const bool bad1 = live && (L1.mode & kInvalid), bad2 = live && (L2.mode & kInvalid);
      const bool bada = live && !(q2 > 0.0 && q2 < INFINITY);
      const unsigned long long nb = __popcll(__ballot(bad1)) + __popcll(__ballot(bad2)) + __popcll(__ballot(bada));
      if (nb && (threadIdx.x & 63) == 0) atomicAdd(nerr, nb);
      const McOrigin o1 = mc_origin(L1, Qs.nqp, P), o2 = mc_origin(L2, Qs.nqp, P);
      double lum = 0.0;
      if (kGW > 1 && !((L1.mode | L2.mode) & (kLowX | kLowQ | kHighQ))) {
        // both lookups inside the grid, read a column group at a
        // time: per step, the kGW values of each lookup that mc_value gives
        // for the group's columns, then the step's terms in request order
        using V = typename VecOf<T, kGW>::type;
        const bool inv1 = L1.mode & kInvalid, inv2 = L2.mode & kInvalid;
        const int ns = __builtin_amdgcn_readfirstlane(sstep[0]);
        for (int s = 0; s < ns; ++s) {
          const int st = __builtin_amdgcn_readfirstlane(sstep[1 + s]);
          if (st == kStepAbsent) {
            const T f1 = inv1 ? (T)NAN : (T)0, f2 = inv2 ? (T)NAN : (T)0;
            lum = fma((double)f1, (double)f2, lum);
            continue;
          }
          const T* g = grid + (st & 0xFFFF);
          // the stencils Q^2 row by Q^2 row (interp_stencil's steps): one
          // row's reads of both lookups in flight at a time
          T f1[kGW], f2[kGW];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            T u1[4][kGW], u2[4][kGW];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              const V q1 = *reinterpret_cast<const V*>(g + o1.x[a] + b * P);
              const V q2v = *reinterpret_cast<const V*>(g + o2.x[a] + b * P);
              __builtin_memcpy(u1[a], &q1, sizeof(V));
              __builtin_memcpy(u2[a], &q2v, sizeof(V));
            }
#pragma unroll
            for (int i = 0; i < kGW; ++i) {
              f1[i] = stencil_step<T>(b, f1[i], u1[0][i], u1[1][i], u1[2][i], u1[3][i], w1, v);
              f2[i] = stencil_step<T>(b, f2[i], u2[0][i], u2[1][i], u2[2][i], u2[3][i], w2, v);
            }
          }
#pragma unroll
          for (int i = 0; i < kGW; ++i) {
            f1[i] = inv1 ? (T)NAN : f1[i];
            f2[i] = inv2 ? (T)NAN : f2[i];
          }
          const int nt = (st >> 16) & 7;
          if (st & kStepOrdered) {
#pragma unroll
            for (int t = 0; t < kGW; ++t)
              if (t < nt) lum = fma((double)f1[t], (double)f2[t], lum);
          } else {
#pragma unroll
            for (int t = 0; t < kGW; ++t)
              if (t < nt) {
                const int e = (st >> (20 + 2 * t)) & 3;
                lum = fma((double)mc_pick<T, kGW>(f1, e), (double)mc_pick<T, kGW>(f2, e), lum);
              }
          }
        }
      } else if (kLdsGrid && kGW == 1 && !((L1.mode | L2.mode) & (kLowX | kLowQ | kHighQ))) {
        // both lookups inside the LDS-staged grid: the values mc_value gives,
        // with both stencils' reads issued together and no branch per point
        // (an invalid point reads the in-bounds stencil at offset 0 and takes
        // NaN); from global memory the 32 loads in flight would spill
        const bool inv1 = L1.mode & kInvalid, inv2 = L2.mode & kInvalid;
        for (int j = 0; j < R; ++j) {
          const int col = __builtin_amdgcn_readfirstlane(scol[j]);
          T f1 = (T)0, f2 = (T)0;
          if (col >= 0) {
            T F1[4][4], F2[4][4];
            const T* g = grid + col;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int b = 0; b < 4; ++b) {
                F1[a][b] = g[o1.x[a] + b * P];
                F2[a][b] = g[o2.x[a] + b * P];
              }
            f1 = interp_stencil<T>(F1, w1, v);
            f2 = interp_stencil<T>(F2, w2, v);
          }
          f1 = inv1 ? (T)NAN : f1;
          f2 = inv2 ? (T)NAN : f2;
          lum = fma((double)f1, (double)f2, lum);
        }
      } else if (!((L1.mode | L2.mode) & (kLowX | kLowQ | kHighQ))) {
        for (int j = 0; j < R; ++j) {
          const int col = scol[j];
          const T f1 = mc_value<T, false>(grid + col, L1, o1, w1, v, P, col, invL01, tb.logt);
          const T f2 = mc_value<T, false>(grid + col, L2, o2, w2, v, P, col, invL01, tb.logt);
          lum = fma((double)f1, (double)f2, lum);
        }
      } else {
        // at least one side extrapolated (rare): the same loop with the
        // extrapolation formulas
        for (int j = 0; j < R; ++j) {
          const int col = scol[j];
          const T f1 = mc_value<T, true>(grid + col, L1, o1, w1, v, P, col, invL01, tb.logt);
          const T f2 = mc_value<T, true>(grid + col, L2, o2, w2, v, P, col, invL01, tb.logt);
          lum = fma((double)f1, (double)f2, lum);
        }
      }
      if (split) {
        acc = live ? lum : 0.0;
        as1 = live ? as : 0.0;
      } else if (live) {
        acc = fma(as, lum, acc);
      }
    }
    if (split) {
      // wave 0 adds the block's terms in the same order: thread t's points in
      // increasing k, then the tree; meanwhile the others take the next block
      __syncthreads();  // wave 0 has read the previous block's terms
      tree[threadIdx.x] = acc;
      tree[kMcFusedBS + threadIdx.x] = as1;
      __syncthreads();
      if (threadIdx.x < 64) {
        double c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          c[u] = 0.0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int e = k * kMcThreads + u * 64 + t;
            c[u] = fma(tree[kMcFusedBS + e], tree[e], c[u]);
          }
        }
        const double v = wave_tree_sum(c[0], c[1], c[2], c[3]);
        if (t == 0) partial[mb] = v;
      }
      continue;
    }
    // the tree of block_tree_sum, per quarter
    double* sh = tree + q * kMcThreads;
    __syncthreads();  // the previous blocks' values have been read
    sh[t] = acc;
    __syncthreads();
    if (t < 64) {
      const double v = wave_tree_sum(sh[t], sh[t + 64], sh[t + 128], sh[t + 192]);
      if (t == 0 && mb < nmb) partial[mb] = v;
    }
  }
}

// LDS bytes of k_mc_fused (grid_elems > 0: the grid staged with row stride P).
static size_t mc_fused_shared_bytes(const MemberDev& m, const AlphasDev& A, int64_t grid_elems, bool f32,
                                    McTables staged) {
  return (staged == kMcAll ? (size_t)m.tbl_bytes : 0) + (size_t)mc_alphas_bytes(A, staged) + kMcFusedBS * 8 +
         (2 * kMaxReq + 4) * 4 + (size_t)grid_elems * (f32 ? 4 : 8);
}

template <typename T>
hipError_t launch_mc_fused(const MemberDev& m, const ReqCols& rc, const AlphasDev& A, const double* x1,
                           const double* x2, const double* q2, int64_t n, double* partial, double* sum_out,
                           unsigned long long* nerr, double invL01, int n_cu, hipStream_t s) {
  const int64_t np = mc_partials(n);
  if (np > 0) {
    constexpr int kGW = sizeof(T) == 4 ? 4 : 1;  // column groups in FP32 only
    const int Pg = (m.P + kGW - 1) & ~(kGW - 1);
    const int64_t rows = m.rows;
    const bool f32 = sizeof(T) == 4;
    // grid in LDS in column groups, else in LDS with stride P, else in global
    // memory; with each, as many of the tables beside it as fit.  From global
    // memory the groups' rows come one after another, which a few waves wait for
    // longer than for single columns (13 columns, 64 points 45.2 against 43.2 us,
    // 128 36.6 and 40.2; 5 columns, 256 points 32.5 and 29.2, 512 39.8 and 42.1)
    const bool few = n * rc.n <= 1500;
    struct Form {
      decltype(&k_mc_fused<T, true, kGW>) kernel;
      int64_t elems;
      McTables staged;
    };
    const Form forms[] = {{&k_mc_fused<T, true, kGW, kMcAll>, rows * Pg, kMcAll},
                          {&k_mc_fused<T, true, kGW, kMcAlphas>, rows * Pg, kMcAlphas},
                          {&k_mc_fused<T, true, kGW, kMcInPlace>, rows * Pg, kMcInPlace},
                          {&k_mc_fused<T, true, 1, kMcAll>, rows * m.P, kMcAll},
                          {&k_mc_fused<T, true, 1, kMcAlphas>, rows * m.P, kMcAlphas},
                          {&k_mc_fused<T, true, 1, kMcInPlace>, rows * m.P, kMcInPlace},
                          {few ? &k_mc_fused<T, false, 1, kMcAll> : &k_mc_fused<T, false, kGW, kMcAll>, 0, kMcAll},
                          {&k_mc_fused<T, false, kGW, kMcAlphas>, 0, kMcAlphas}};
    // One block of points per workgroup, its four points per thread over the
    // four quarters, when that takes fewer rounds than four blocks per
    // workgroup: rounds of 1024 points on the slots of the chip (300007 points,
    // 293 blocks: 2 rounds instead of 4, FP32 55 -> 38 us then, 32 now; 1e6 points:
    // 4 either way, and then the barrier per round costs 3 %, 91 against 94 us).
    // It needs a second tree, and is then worth more than tables in LDS or
    // column groups (FP32, 13 columns, 3e5 points: 58 us against 106).
    auto rounds = [&](size_t bytes, int per_wg) {
      const int64_t slots = (int64_t)n_cu * max(1, (int)(160 * 1024 / bytes));
      return ((np + per_wg - 1) / per_wg + slots - 1) / slots * per_wg;
    };
    constexpr size_t kTree = kMcFusedBS * 8;
    const Form* form = nullptr;
    size_t shm = 0;
    int split = 0;
    for (const Form& f : forms) {
      const size_t b = mc_fused_shared_bytes(m, A, f.elems, f32, f.staged);
      if (b > 160 * 1024) continue;  // the last always fits: at most 28 KB of alpha_s table
      if (!form) {
        form = &f;
        shm = b;
      }
      // a grid in LDS comes first; in FP32 and with few blocks not before four
      // quarters on one (50 x 56 x 13, 10^5 points: 101 us, from global memory
      // 79, and with 5 % of the points outside 207 and 96; 2 10^5 points: 103 and
      // 108; FP64, 50 x 33 x 11, 10^5 points: 86 and 198)
      if (form->elems && !f.elems && !(kGW > 1 && 2 * np <= n_cu)) break;
      if (b + kTree <= 160 * 1024 && rounds(b + kTree, 1) < rounds(b, 4)) {
        form = &f;
        shm = b + kTree;
        split = 1;
        break;
      }
    }
    auto kernel = form->kernel;
    const void* fn = reinterpret_cast<const void*>(kernel);
    hipError_t e = allow_dynamic_lds(fn, shm);
    if (e != hipSuccess) return e;
    const int per_cu = max(1, (int)(160 * 1024 / shm));
    const int64_t nb = min(split ? np : (np + 3) / 4, (int64_t)n_cu * per_cu);
    hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(kMcFusedBS), shm, s, m, rc, A, x1, x2, q2, n, partial, nerr,
                       invL01, split);
  }
  hipLaunchKernelGGL(k_mc_final, dim3(1), dim3(kMcThreads), 0, s, partial, np, sum_out);
  return hipGetLastError();
}
template hipError_t launch_mc_fused<double>(const MemberDev&, const ReqCols&, const AlphasDev&, const double*,
                                            const double*, const double*, int64_t, double*, double*,
                                            unsigned long long*, double, int, hipStream_t);
template hipError_t launch_mc_fused<float>(const MemberDev&, const ReqCols&, const AlphasDev&, const double*,
                                           const double*, const double*, int64_t, double*, double*,
                                           unsigned long long*, double, int, hipStream_t);

template hipError_t launch_mc_sum<double>(const double*, const double*, int, const double*, int64_t, double*, double*,
                                          hipStream_t);
template hipError_t launch_mc_sum<float>(const float*, const float*, int, const double*, int64_t, double*, double*,
                                         hipStream_t);

}  // namespace pdfmi

namespace pdfmi {

// ---------------------------------------------------------------------------------------
// Batched evaluation of many requests over many members (the paper's
// multi-member evaluation of section 4.3): one persistent launch in which
// each workgroup takes a first tile of its own, then repeatedly the next
// one from a counter, stages that tile's grid (and location tables) in
// LDS when it differs from the one already staged, and runs the same per-wave
// tile pipeline as k_xfxq2.  A wave's first points are loaded before the
// staging and the next ones before the current are evaluated.  The first tiles
// go to the 8 XCDs, which take workgroups in turn, in contiguous runs: a member's
// rows are then read into one L2 and not into eight (100 members x 15000 points,
// 13 columns of 1.3 MB a member, FP64: 347 us with the tile of the workgroup's
// index, 259 with the first tile from the counter too, 236 so).  Every wave
// reaches the exit once the counter passes the tile count.
//
// Runs of one plan on different streams may overlap, and each has to have
// evaluated every tile by its own end, so a run has its counter to itself (with
// one per plan, the tiles taken by one run would be left out by the other).
// The last workgroup to leave clears the counter and tells the host, which
// then gives it to another run; a kernel before each run that clears it takes
// about 4 us, an event recorded after it 6.  A run without a counter, because
// all are in use, deals the tiles out in a fixed order (514 us against 490 for
// the 101-member plan).
//
// In FP32 with the grid in LDS, a request of up to kCompactCols different
// flavours (BatchReq::layout >= 0) is staged compacted: rows of kCompactCols
// floats holding the requested columns in request order.  Its outputs are
// then walked in groups of four columns (two, one for the smallest requests)
// with one LDS read per group and stencil knot, whatever the order of the
// request: what bounded the kernel were the conflicts of one 4-byte read per
// (flavour, knot) from random rows (101 members, 200 requests, 1.2e8 values:
// 705 us, 541 with this layout).  Rows of 48 bytes start on every 16-byte bank slot, and
// a compile-time stride lets the four Q^2 rows use immediate offsets.
// One workgroup of 1024 threads per compute unit; where the grids are read from
// global memory and there are no more tiles of 512 points than two workgroups
// of half the size per compute unit, those (kBatchHalf), so that a plan of few
// points spreads over more of them (100 members x 2415 points, FP64: tiles of
// 512 points on 500 of 512 slots instead of 200 tiles of up to 2048 on 256).
// With more points they are the slower ones, as twice as many tiles, and so
// members, share the caches (100 requests of 30000 points, 100 members of 1.3
// MB, FP64, one column: 576 us where 1024 threads took 475).
// Grids that fit LDS only without four of the 16 waves' records get workgroups
// of 12 (kBatchSmall).
constexpr int kCompactRowB = kCompactCols * 4;

// kCounted: more tiles than workgroups (without it the arguments of the counter alone cost 0.3 us a run).
template <typename T, bool kLdsGrid, bool kLdsTables, bool kCounted, int kBS>
__global__ __launch_bounds__(kBS) __attribute__((amdgpu_waves_per_eu(4))) void k_batched(const BatchReq* __restrict__ reqs, const int* __restrict__ cols,
                                                      const BatchTile* __restrict__ tiles, int ntiles,
                                                      const MemberDev* __restrict__ members,
                                                      const double* __restrict__ invL01s, RunSlot* slot,
                                                      unsigned* done, unsigned run,
                                                      unsigned long long* __restrict__ nerr, int max_tbl,
                                                      int vector_cols) {
  static_assert(kLdsTables || !kLdsGrid, "a staged grid needs staged tables");
  constexpr int kWaves = kBS / kWave;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_tile;
  unsigned char* stbl = smem;                                              // [max_tbl] if staged
  int* scol = reinterpret_cast<int*>(smem + (kLdsTables ? max_tbl : 0));  // [kMaxReq]
  unsigned char* srec = reinterpret_cast<unsigned char*>(scol + kMaxReq);  // per-wave records
  T* sgrid = reinterpret_cast<T*>(srec + kWaves * wave_record_bytes<T>());
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  unsigned char* rec = srec + wv * wave_record_bytes<T>();
  int staged_member = -1, staged_layout = -1;  // layouts are >= 0, or <= -2 for all columns of a member
  // the first tile is the workgroup's own, the others come from the counter
  const int per = (int)(gridDim.x >> 3), rest = (int)(gridDim.x & 7), xcd = (int)(blockIdx.x & 7);
  const int t0 = xcd * per + min(xcd, rest) + (int)(blockIdx.x >> 3);
  for (int t = t0; t < ntiles; t = __builtin_amdgcn_readfirstlane(s_tile)) {
    const BatchTile tl = tiles[t];
    const BatchReq rq = reqs[tl.req];
    const MemberDev& m = members[rq.member];
    const T* __restrict__ gvals = member_values<T>(m);
    const uint32_t gbytes = (uint32_t)((sizeof(T) == 8 ? m.elems64 : m.elems32) * (int64_t)sizeof(T));
    // what the staged grid holds: a compacted layout, or all columns of a member
    const bool compact = kLdsGrid && sizeof(T) == 4 && vector_cols && rq.layout >= 0;
    const int layout = compact ? rq.layout : -2 - rq.member;
    const int* rcols = cols + rq.col_off;
    // the points of a pass are loaded before the one before it is evaluated, the first before the staging
    const PDFMI_GLOBAL double* px = (const PDFMI_GLOBAL double*)rq.x + tl.start;
    const PDFMI_GLOBAL double* pq = (const PDFMI_GLOBAL double*)rq.q2 + tl.start;
    double xn = 0.0, qn = 0.0;
    if (wv * kWave + lane < tl.count) {
      xn = px[wv * kWave + lane];
      qn = pq[wv * kWave + lane];
    }
    if constexpr (kLdsTables)
      if (rq.member != staged_member) stage_copy<kBS>(stbl, m.tables, m.tbl_bytes);
    if constexpr (kLdsGrid)
      if (layout != staged_layout) {
        if (compact) {
          float* g = reinterpret_cast<float*>(sgrid);
          stage_columns<kBS, kCompactCols>(g, m.v32, m.rows, m.P, m.P32, rcols + rq.R);
          for (int j = 0; j < rq.R; ++j)
            if (rcols[j] < 0)
              for (int i = threadIdx.x; i < m.rows; i += kBS) g[i * kCompactCols + j] = 0.0f;
        } else {
          stage_copy<kBS>(sgrid, gvals, (int64_t)gbytes);
        }
      }
    for (int i = threadIdx.x; i < rq.R; i += kBS) scol[i] = rcols[i];
    __syncthreads();
    staged_member = rq.member;
    staged_layout = layout;
    const Tables tb = tables_at(kLdsTables ? stbl : m.tables, m);
    const double invL01 = invL01s[rq.member];
    T* out = reinterpret_cast<T*>(rq.out);
    int nslow = 0;
    for (int w0 = wv * kWave; w0 < tl.count; w0 += kWaves * kWave) {
      const int64_t pbeg = tl.start + w0;
      const int tp = min(kWave, tl.count - w0);
      constexpr int G = 16 / sizeof(T);
      const double xv = xn, qv = qn;
      xn = qn = 0.0;
      const int nxt = w0 + kWaves * kWave + lane;
      if (nxt < tl.count) {
        xn = px[nxt];
        qn = pq[nxt];
      }
      if constexpr (kLdsGrid && sizeof(T) == 4) {
        if (compact) {
          auto tile = [&](auto group) {
            wave_tile<T, true, decltype(group)::value, false, false, kCompactRowB, true>(
                m, tb, scol, rq.R, sgrid, gvals, gbytes, xv, qv, tp, out + pbeg * rq.R, nerr, invL01, rec, nslow,
                lane, kNoAlphas, AsView{});
          };
          if (rq.R > 2)
            tile(std::integral_constant<int, 4>{});
          else if (rq.R == 2)
            tile(std::integral_constant<int, 2>{});
          else
            tile(std::integral_constant<int, 1>{});
          continue;
        }
      }
      if (vector_cols && rq.all_cols && rq.R >= G)
        wave_tile<T, kLdsGrid, G>(m, tb, scol, rq.R, sgrid, gvals, gbytes, xv, qv, tp, out + pbeg * rq.R, nerr,
                                  invL01, rec, nslow, lane, kNoAlphas, AsView{});
      else if (kLdsGrid && sizeof(T) == 4 && m.P32 == 12)  // 9-12 stored flavours in FP32: 48-byte rows
        wave_tile<T, kLdsGrid, 1, false, !kLdsGrid, 48>(m, tb, scol, rq.R, sgrid, gvals, gbytes, xv, qv, tp,
                                                        out + pbeg * rq.R, nerr, invL01, rec, nslow, lane, kNoAlphas,
                                                        AsView{});
      else
        wave_tile<T, kLdsGrid, 1>(m, tb, scol, rq.R, sgrid, gvals, gbytes, xv, qv, tp, out + pbeg * rq.R, nerr,
                                  invL01, rec, nslow, lane, kNoAlphas, AsView{});
    }
    if (nslow > 0) {
      const SlowRec<T>* q = reinterpret_cast<const SlowRec<T>*>(rec + kWave * sizeof(PointRec<T>));
      const T* g0 = kLdsGrid ? sgrid : gvals;
      if (compact)
        finish_slow<T, !kLdsGrid, true>(q, nslow, rq.R, scol, g0, kCompactCols, invL01, tb.logt, lane);
      else
        finish_slow<T, !kLdsGrid>(q, nslow, rq.R, scol, g0, sizeof(T) == 8 ? m.P64 : m.P32, invL01, tb.logt, lane);
    }
    if constexpr (!kCounted) break;  // no more tiles than workgroups
    if (threadIdx.x == 0) s_tile = slot ? (int)(gridDim.x + atomicAdd(&slot->taken, 1u)) : t + (int)gridDim.x;
    __syncthreads();  // the next tile is known, and every wave has left this one's LDS
  }
  // Relaxed atomics, in order because each waits for the one before: what this
  // workgroup took of the count it has seen before it leaves.  (With acquire
  // and release every workgroup writes its L2 back: 6 us a run.)
  if (kCounted && slot && threadIdx.x == 0 &&
      __hip_atomic_fetch_add(&slot->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
    // no workgroup of this run takes another tile
    __hip_atomic_store(&slot->taken, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot->left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(done, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Location tables are staged when the largest member's fit (always when the
// grid is staged too).
static bool batch_tables(bool lds, int max_tbl) { return lds || (size_t)max_tbl <= kMaxLdsTables; }

size_t batch_shared_bytes(int max_tbl, bool f32, bool lds, int block) {
  return (batch_tables(lds, max_tbl) ? (size_t)max_tbl : 0) + kMaxReq * 4 +
         (block / kWave) * (f32 ? wave_record_bytes<float>() : wave_record_bytes<double>());
}

// Kernel node parameters of one batched run (used for direct launches and for building a hipGraph).

template <typename T, bool kCounted>
static const void* batch_fn(bool lds, bool tables, int block) {
  if (lds)
    return block == kBatchThreads ? reinterpret_cast<const void*>(&k_batched<T, true, true, kCounted, kBatchThreads>)
                                  : reinterpret_cast<const void*>(&k_batched<T, true, true, kCounted, kBatchSmall>);
  if (!kCounted && block == kBatchHalf)
    return tables ? reinterpret_cast<const void*>(&k_batched<T, false, true, false, kBatchHalf>)
                  : reinterpret_cast<const void*>(&k_batched<T, false, false, false, kBatchHalf>);
  return tables ? reinterpret_cast<const void*>(&k_batched<T, false, true, kCounted, kBatchThreads>)
                : reinterpret_cast<const void*>(&k_batched<T, false, false, kCounted, kBatchThreads>);
}

BatchLaunch batch_launch_params(bool f32, bool lds, int max_tbl, int64_t max_elems, int n_cu, int ntiles, int block) {
  BatchLaunch L{};
  L.shm = batch_shared_bytes(max_tbl, f32, lds, block) + (lds ? (size_t)max_elems * (f32 ? 4 : 8) : 0);
  const bool tables = batch_tables(lds, max_tbl);
  L.block = (unsigned)block;
  const int64_t g = min((int64_t)ntiles, (int64_t)n_cu * (block == kBatchHalf ? 2 : 1));
  L.grid = (unsigned)max((int64_t)1, g);
  L.counted = ntiles > (int)L.grid;
  L.main_fn = L.counted ? (f32 ? batch_fn<float, true>(lds, tables, block) : batch_fn<double, true>(lds, tables, block))
                        : (f32 ? batch_fn<float, false>(lds, tables, block) : batch_fn<double, false>(lds, tables, block));
  return L;
}

hipError_t batch_prepare(const BatchLaunch& L) {
  return allow_dynamic_lds(L.main_fn, L.shm);
}

hipError_t batch_launch(const BatchLaunch& L, void** args, hipStream_t s) {
  return hipLaunchKernel(L.main_fn, dim3(L.grid), dim3(L.block), args, L.shm, s);
}

}  // namespace pdfmi
