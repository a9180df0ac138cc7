// Device functions of the interpolation (shared by the interpolation,
// batched and surrogate kernels): knot search, Hermite stencil weights,
// point location, in-grid stencil sum and the extrapolation formulas.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "pdfmi_dev.h"

#define PDFMI_GLOBAL __attribute__((address_space(1)))  // a pointer read from memory is global, not generic

namespace pdfmi {

// Point-location tables as a kernel reads them: from LDS (staged copy of the
// member's table block) or from global memory.
struct Tables {
  const double* knots;
  const CellCoef* cells;
  const QCell* qcells;
  const short* hints;
  const SubDesc* subs;
  const LogEntry* logt;
};

__device__ __forceinline__ Tables tables_at(const unsigned char* base, const MemberDev& m) {
  return Tables{reinterpret_cast<const double*>(base), reinterpret_cast<const CellCoef*>(base + m.cells_off),
                reinterpret_cast<const QCell*>(base + m.qcells_off),
                reinterpret_cast<const short*>(base + m.hints_off),
                reinterpret_cast<const SubDesc*>(base + m.subs_off),
                reinterpret_cast<const LogEntry*>(base + m.logt_off)};
}

__device__ __forceinline__ int high_word(double v) { return __double2hiint(v); }

// ln v by table, by the method of the log function of Arm's Optimized Routines
// (MIT, or Apache-2.0 with LLVM exception): reduction by the high word to
// v = 2^k z, z in [0.6875, 1.375); z in interval i of 128 with c_i near its
// middle; r = z / c_i - 1 by one fma, |r| <= 2^-7;
// ln v = k ln 2 + ln c_i + log1p(r).  The two intervals next to 1 have c = 1,
// so small logarithms keep their relative precision; ln 2 is split so that
// k ln 2's high part is exact, the error of its sum with ln c_i is carried,
// and the c_i are chosen so that ln c_i is a double to about 1/64 ulp.  The
// table is made by make_log_table, log1p is its plain series.  Error
// against long double: rms 0.28-0.31 ulp, as the correctly rounded result's,
// at most 1 ulp.  About 25 instructions and one 16-byte table read; with the
// library function (about 100) alpha_s of 1e7 points took 86 us, now 37.
__device__ __forceinline__ double normal_log(double v, int kadd, const LogEntry* __restrict__ t) {
  const int hi = high_word(v);
  const int off = hi - kLogOrigin;
  const LogEntry e = t[(off >> 13) & (kLogEntries - 1)];
  const double z = __hiloint2double(hi - (off & (int)0xfff00000), __double2loint(v));
  const double r = fma(z, e.inv, -1.0);
  double q = fma(r, -1.0 / 8.0, 1.0 / 7.0);
  q = fma(r, q, -1.0 / 6.0);
  q = fma(r, q, 1.0 / 5.0);
  q = fma(r, q, -1.0 / 4.0);
  q = fma(r, q, 1.0 / 3.0);
  q = fma(r, q, -0.5);
  const double k = (double)((off >> 20) + kadd);
  const double a = k * 0x1.62e42fefa3800p-1;  // high part of ln 2, 11 trailing zero bits
  const double s = a + e.log;
  const double err = e.log - (s - a);
  return s + (r + fma(r * r, q, fma(k, 0x1.ef35793c76730p-45, err)));
}
// Arguments that are not positive normal numbers: subnormals scaled, the rest as the library function.
__device__ __forceinline__ double fast_log(double v, const LogEntry* __restrict__ t) {
  double l = normal_log(v, 0, t);
  if ((unsigned)(high_word(v) - 0x00100000) >= 0x7fe00000u)  // not a positive normal number
    l = v == 0.0 ? -INFINITY : (v > 0.0 && v < INFINITY ? normal_log(v * 0x1p54, -54, t) : (v > 0.0 ? v : NAN));
  return l;
}

// Largest i in [0, n-2] with t[i] <= v, 0 if t[0] > v (t strictly increasing).
__device__ __forceinline__ int find_cell_binary(const double* __restrict__ t, int n, double v) {
  const int last = n - 2;
  int i = 0;
  int step = last > 0 ? (1 << (31 - __builtin_clz((unsigned)last))) : 0;
  for (; step > 0; step >>= 1) {
    const int j = i + step;
    if (j <= last && t[j] <= v) i = j;
  }
  return i;
}

// The same index from the table's bucket hints (see HintAxis): one hint read,
// then two independent knot comparisons.  Knot i + 2 may lie one past the
// table (whatever follows it in the block is read): the index is then at
// least n-2 already and the comparison changes nothing.  Any v (NaN, <= 0)
// gives an index in range.
__device__ __forceinline__ int find_cell(const double* __restrict__ t, int n, double v, const HintAxis& h,
                                         const short* __restrict__ hints) {
  if (h.off < 0) return find_cell_binary(t, n, v);
  const int b = min(max((int)((unsigned)high_word(v) >> h.shift) - h.key0, 0), h.n - 1);
  const int i = hints[h.off + b];
  return min(i + (t[i + 1] <= v ? 1 : 0) + (t[i + 2] <= v ? 1 : 0), n - 2);
}

// Hermite weights of knots i-1..i+2 at cell parameter u (see CellCoef).  The
// basis in factored form: 1 - u is exact, so every basis value keeps its
// relative precision near u = 0 and u = 1 (the expanded forms cancel there,
// leaving absolute errors of one ulp that the large weights of a cell next to
// a much narrower one magnify).
template <typename T>
__device__ __forceinline__ void hermite_weights(double u64, const CellCoef& c, T r[4]) {
  const T u = (T)u64;
  const T w = (T)1 - u;
  const T u2 = u * u, w2 = w * w;
  const T h10 = u * w2, h11 = -(w * u2);
  const T hl = (T)c.hl, hr = (T)c.hr, el = (T)c.el, er = (T)c.er;
  r[0] = -(hl * h10);
  r[1] = fma(w2, fma((T)2, u, (T)1), fma(hl - el, h10, -(er * h11)));   // h00 + ...
  r[2] = fma(u2, fma((T)-2, u, (T)3), fma(er - hr, h11, el * h10));     // h01 + ...
  r[3] = hr * h11;
}

// Cell parameter of v, exactly 0 at the cell's first knot.
__device__ __forceinline__ double cell_u(double v, double t0, double l, double invD) {
  return v == t0 ? 0.0 : l * invD;
}

// Entry i of a table of E (multiplication in 24 bits: full rate).
template <typename E>
__device__ __forceinline__ const E& entry(const void* base, int i) {
  return *reinterpret_cast<const E*>(static_cast<const unsigned char*>(base) +
                                     __umul24((unsigned)i, (unsigned)sizeof(E)));
}

// The alpha_s table as a kernel reads it (the block staged in LDS; logt is
// the block's own or an equal copy) and where a fused evaluation writes
// alpha_s: out == nullptr means no alpha_s output.
struct AsView {
  const unsigned char* base;
  const LogEntry* logt;
  double* out;
};

// alpha_s at one Q^2: cubic Hermite in ln Q^2 inside a segment, constant
// outside the knots; NaN for Q^2 <= 0 or non-finite.
__device__ __forceinline__ double alphas_point(const AlphasDev& A, const AsView& av, double q2) {
  const double* sk = reinterpret_cast<const double*>(av.base);
  const int i = find_cell(sk, A.ncell + 1, q2, A.h, reinterpret_cast<const short*>(av.base + A.hints_off));
  const AsCell& c = entry<AsCell>(av.base + A.cells_off, i);
  const double u = cell_u(q2, c.t0, fast_log(q2 * c.inv_t0, av.logt), c.invD), w = 1.0 - u, u2 = u * u;
  // f0 + h01 df + h10 d0 + h11 d1 (h00 = 1 - h01)
  double acc = c.f0 + fma(u2 * fma(-2.0, u, 3.0), c.df, (u * w) * fma(w, c.d0, -(u * c.d1)));
  if (!(q2 >= A.q_lo && q2 < A.q_hi)) {
    acc = q2 < A.q_lo ? A.a_lo : A.a_hi;
    if (!(q2 > 0.0 && q2 < INFINITY)) acc = NAN;
  }
  return acc;
}

// Location of a point in a member's grid, in two halves so that points that
// share Q^2 (the two lookups of a Monte-Carlo point) locate it once.  Every
// kernel uses these functions, so the fused and the separate evaluations agree
// bit for bit.
//
// The stencil of a point: Q^2 knots sq .. sq+3 (kept inside the sub-grid) with
// weights v; x knots ix-1 .. ix+2 with weights w, where a knot outside the
// table is replaced by its neighbour ix or ix+1 (its weight is 0).  In rows of
// P values the four x knots start at row, row + s1, + nqp, + s3 (each added to
// the one before; s1 and s3 are nqp or 0).
template <typename T>
struct QLoc {
  T v[4];
  int row, nqp, kiq, d;
  double u;  // cell parameter
  double r;  // Q^2 / t0
};

template <typename T>
__device__ __forceinline__ QLoc<T> locate_q(const MemberDev& m, const Tables& tb, double q2) {
  const QCell& c = entry<QCell>(tb.qcells, find_cell(tb.knots + m.qk_off, m.nqk, q2, m.qh, tb.hints));
  QLoc<T> Q;
  Q.row = c.row;
  Q.nqp = c.nqp;
  Q.kiq = c.kiq;
  Q.d = c.d;
  Q.r = q2 * c.c.inv_t0;
  Q.u = cell_u(q2, c.c.t0, fast_log(Q.r, tb.logt), c.c.invD);
  if (q2 == m.qmax) Q.u = 1.0;
  T r[4];
  hermite_weights<T>(Q.u, c.c, r);
  // r[0] (left end) and r[3] (right end) are 0 where the shift would lose them
  const bool lo = c.d == 0, hi = c.d == 2;
  Q.v[0] = lo ? r[1] : (hi ? (T)0 : r[0]);
  Q.v[1] = lo ? r[2] : (hi ? r[0] : r[1]);
  Q.v[2] = lo ? r[3] : (hi ? r[1] : r[2]);
  Q.v[3] = lo ? (T)0 : (hi ? r[2] : r[3]);
  return Q;
}

struct PointLoc {
  int mode;      // 0 inside the grid; else region bits | kXHigh | (anchor row << 8) for high Q^2
  int ix;
  int row, s1, s3;  // stencil rows (see above; nqp from the QLoc)
  double p0, p1; // extrapolation parameters
};

// Completes the location of (x, q2) given Q = locate_q(q2): x weights w, and
// for points outside the grid the region and its parameters.  v: the Q^2
// weights the point uses (Q.v inside).
template <typename T>
__device__ __forceinline__ PointLoc locate_x(const MemberDev& m, const Tables& tb, const QLoc<T>& Q, double x,
                                             double q2, T w[4], T v[4]) {
  PointLoc L;
  int nx = m.nx, xk = m.xk_off, xc = m.xc_off;
  HintAxis xh = m.xh;
  if (!m.shared_x) {
    const SubDesc S = tb.subs[Q.kiq >> 16];
    nx = S.nx;
    xk = S.xk_off;
    xc = S.xc_off;
    xh = S.xh;
  }
  const int ix = find_cell(tb.knots + xk, nx, x, xh, tb.hints);
  const CellCoef& c = entry<CellCoef>(tb.cells, xc + ix);
  const double u = cell_u(x, c.t0, fast_log(x * c.inv_t0, tb.logt), c.invD);
  hermite_weights<T>(u, c, w);
#pragma unroll
  for (int b = 0; b < 4; ++b) v[b] = Q.v[b];
  L.mode = 0;
  L.p0 = 0.0;
  L.p1 = 0.0;
  L.ix = ix;
  L.s1 = ix > 0 ? Q.nqp : 0;
  L.s3 = ix < nx - 2 ? Q.nqp : 0;
  L.row = Q.row + (int)__umul24((unsigned)ix, (unsigned)Q.nqp) - L.s1;
  if (!(x >= m.xmin && x < m.xmax && q2 >= m.qmin && q2 <= m.qmax)) {
    if (x == m.xmax) {  // the last knot: exact weights
      w[0] = w[1] = w[3] = (T)0;
      w[2] = (T)1;
    }
    const bool valid = (x > 0.0) && (x <= m.xmax) && (q2 > 0.0) && (q2 < INFINITY);
    const bool lowx = x < m.xmin, lowq = q2 < m.qmin, highq = q2 > m.qmax;
    if (!valid) {
      L.mode = kInvalid;
    } else if (lowx || lowq || highq) {
      // one logarithm per axis whatever the region: below x_0 the cell is the
      // first one and u = ln(x/x_0) / ln(x_1/x_0) is the continuation
      // parameter itself; above the last Q^2 knot
      // Q.u - 1 = ln(Q^2/q_n-1) / ln(q_n-1/q_n-2), and the stencil row of q_n-2 is Q.d
      L.mode = (lowx ? kLowX : 0) | (lowq ? kLowQ : 0) | (highq ? kHighQ | (Q.d << 8) : 0) | (x > 0.9 ? kXHigh : 0);
      if (lowq) L.p0 = Q.r; else if (highq) L.p0 = Q.u - 1.0; else L.p0 = u;
      if (lowx && (lowq || highq)) L.p1 = u;
    }
    if (!valid || lowx)
#pragma unroll
      for (int a = 0; a < 4; ++a) w[a] = (T)0;
    if (!valid || lowq || highq)
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = (T)0;
  }
  return L;
}

template <typename T>
__device__ __forceinline__ const T* member_values(const MemberDev& m);
template <>
__device__ __forceinline__ const double* member_values<double>(const MemberDev& m) { return m.v64; }
template <>
__device__ __forceinline__ const float* member_values<float>(const MemberDev& m) { return m.v32; }

// In-grid value of one column from its gathered 4x4 stencil: the x-direction
// weights on each of the four Q^2 rows, then the Q^2-direction weights.
// stencil_step adds Q^2 row b (its four x-knot values f0..f3) to the running
// sum acc; interp_stencil is the four steps in order, and a caller that
// gathers the stencil row by row may take the steps itself with the same
// result.
template <typename T>
__device__ __forceinline__ T stencil_step(int b, T acc, T f0, T f1, T f2, T f3, const T w[4], const T v[4]) {
  T g = w[0] * f0;
  g = fma(w[1], f1, g);
  g = fma(w[2], f2, g);
  g = fma(w[3], f3, g);
  return b == 0 ? v[0] * g : fma(v[b], g, acc);
}

template <typename T>
__device__ __forceinline__ T interp_stencil(const T F[4][4], const T w[4], const T v[4]) {
  T acc = (T)0;
#pragma unroll
  for (int b = 0; b < 4; ++b) acc = stencil_step<T>(b, acc, F[0][b], F[1][b], F[2][b], F[3][b], w, v);
  return acc;
}

// Two-anchor continuation from f0 by the parameter s (log-linear when both
// anchors exceed 1e-3); `from` is the anchor the parameter counts from.
// Powers are exp(b ln a): the bases are positive ratios, and a few ulps of
// exp and log stay far inside the FP64 parity bound.
__device__ __forceinline__ double continued(double from, double f0, double f1, double s, const LogEntry* lt) {
  return (f0 > 1e-3 && f1 > 1e-3) ? from * exp(s * fast_log(f1 / f0, lt)) : from + s * (f1 - f0);
}

// Extrapolated value of one column (rare path, FP64 combination).  f points at
// the column's entry of the stencil's first row; s1, sa, s3 are the steps
// between its x knots and Pp the stride between Q^2 knots (elements).  Only the
// anchor knots the formula needs are read:
//   x below x_min only:     a0, a1 = rows x_0, x_1 interpolated in Q^2
//   Q^2 outside, x inside:  a0, a1 = the two anchor Q^2 rows interpolated in x
//   corners:                x_0, x_1 on the lower and on the upper anchor row,
//                           continued in x to a0 and a1
// (below x_min the cell is the first one: x_0 and x_1 are the stencil's
// second and third x knot).  Then from a0, a1: the two-anchor continuation, or
// below Q^2_min f0 r^(gamma r + 1 - r) with gamma from the first two Q^2 knots.
// Lanes of one wave hold points of different regions: the regions share one
// gather of four anchor pairs, one division, one exponential and at most two
// logarithms instead of a branch each.
// A call (its arguments in registers): inlined, it would cost the callers'
// common path registers.  kGlobal: f is in global memory.
template <typename T, bool kGlobal>
static __device__ __noinline__ double extrap_entry(const T* fp, int s1, int sa, int s3, int Pp, int mode, T w0, T w1, T w2,
                                                   T w3, T v0, T v1, T v2, T v3, double p0, double p1, double invL01,
                                                   const LogEntry* lt) {
  using Ptr = std::conditional_t<kGlobal, const PDFMI_GLOBAL T*, const T*>;
  const Ptr f = (Ptr)fp;
  const bool lowx = mode & kLowX, lowq = mode & kLowQ, highq = mode & kHighQ;
  const bool xonly = lowx && !(lowq || highq), corner = lowx && !xonly;
  const int r0 = lowq ? 0 : ((mode >> 8) & 3) * Pp;  // lower anchor row
  // terms of a0 (offset, weight); a1 has the same at `step`
  const int o0 = xonly ? s1 : (corner ? s1 + r0 : r0);
  const int o1 = xonly ? s1 + Pp : (corner ? o0 : r0 + s1);
  const int o2 = xonly ? s1 + 2 * Pp : (corner ? o0 : r0 + s1 + sa);
  const int o3 = xonly ? s1 + 3 * Pp : (corner ? o0 : r0 + s1 + sa + s3);
  const int step = lowx ? sa : Pp;
  const double c0 = (double)(xonly ? v0 : w0), c1 = (double)(xonly ? v1 : w1);
  const double c2 = (double)(xonly ? v2 : w2), c3 = (double)(xonly ? v3 : w3);
  const double f00 = (double)f[o0], f10 = (double)f[o0 + step];
  double a0 = c0 * f00, a1 = c0 * f10;
  a0 = fma(c1, (double)f[o1], a0);
  a1 = fma(c1, (double)f[o1 + step], a1);
  a0 = fma(c2, (double)f[o2], a0);
  a1 = fma(c2, (double)f[o2 + step], a1);
  a0 = fma(c3, (double)f[o3], a0);
  a1 = fma(c3, (double)f[o3 + step], a1);
  if (corner) {
    a0 = continued(f00, f00, f10, p1, lt);
    const double f01 = (double)f[o0 + Pp], f11 = (double)f[o0 + Pp + step];
    a1 = continued(f01, f01, f11, p1, lt);
  }
  const double from = highq ? a1 : a0;
  const double least = lowq ? 1e-5 : 1e-3;
  double val = lowq ? a0 * p0 : from + p0 * (a1 - a0);
  if (a0 > least && a1 > least && !(lowq && (mode & kXHigh))) {
    const double lr = fast_log(a1 / a0, lt);
    double e = p0 * lr;
    if (lowq) {
      const double gamma = lr * invL01;
      e = (gamma * p0 + 1.0 - p0) * fast_log(p0, lt);
    }
    val = from * exp(e);
  }
  return val;
}

// Per-point record of a located point, written by one lane and read by
// others: weights and location side by side (80 bytes in FP64, 48 in FP32), so
// that the 9-16 different records one load instruction reads fall in
// different LDS banks.  Locations are bytes: the stencil's first row and the
// steps between its x knots.  All are multiples of 4; bits 0 and 1 of o say
// outside the grid and invalid (the mode of a point outside is kept apart).
template <typename T>
struct PointRec {
  T w[4];
  T v[4];
  int o, s1, sa, s3;
};
constexpr int kRecSlow = 1, kRecInvalid = 2;

// A point outside the grid, kept until enough of them fill a wave.
template <typename T>
struct SlowRec {
  PointRec<T> r;
  double p0, p1;  // extrapolation parameters
  int mode, pad;
  T* out;         // the point's output row
};

template <typename T>
__device__ __forceinline__ void set_stencil(PointRec<T>& r, const QLoc<T>& Q, const PointLoc& L, int rowb) {
  r.o = (int)__umul24((unsigned)L.row, (unsigned)rowb);
  r.sa = (int)__umul24((unsigned)Q.nqp, (unsigned)rowb);
  r.s1 = L.s1 ? r.sa : 0;
  r.s3 = L.s3 ? r.sa : 0;
  if (L.mode) r.o |= L.mode & kInvalid ? kRecInvalid : kRecSlow;
}

// One column of a point outside the grid (kRecSlow) with its mode and
// extrapolation parameters; col0 points at the column's entry of grid row 0.
template <typename T, bool kGlobal>
__device__ __forceinline__ T rec_extrapolate(const PointRec<T>& r, int mode, double p0, double p1, const T* col0,
                                             int Pp, double invL01, const LogEntry* lt) {
  const int es = (int)sizeof(T);
  const T* f = reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(col0) + (r.o & ~3));
  return (T)extrap_entry<T, kGlobal>(f, r.s1 / es, r.sa / es, r.s3 / es, Pp, mode, r.w[0], r.w[1], r.w[2], r.w[3], r.v[0],
                                     r.v[1], r.v[2], r.v[3], p0, p1, invL01, lt);
}

}  // namespace pdfmi
