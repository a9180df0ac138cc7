// MLP surrogate of one member's PDFs (growth path of the interpolation
// library): (ln x, ln Q^2) -> all stored flavours, 2 -> 64 -> 64 -> 64 -> 16
// (outputs beyond the stored columns are padding), tanh hidden activations,
// FP32 master weights trained with Adam.
//
// Arithmetic: the first layer (two inputs) in FP32 on the vector ALUs;
// layers 2-4 on the matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation) with every operand carried as a BF16 pair (value = hi + lo,
// lo = bf16(value - hi)) and each product formed as hi*hi + lo*hi + hi*lo:
// about 16 significant bits per operand, where single BF16 operands (8 bits)
// left the network's relative error near 1e-3.  The backward pass multiplies
// BF16 signals with the hi halves.
//
// The network predicts y_c = xf_c / E_c(x), where E_c is a signed cubic
// Hermite envelope in ln x through the grid value of largest magnitude at
// each x knot (it follows the x dependence, sign changes included, so the
// targets are smooth and O(1)).  Training uses only samples inside the
// network's domain; inference falls back to the FP32 interpolator outside
// the grid and in the first/last x or Q^2 cell of a sub-grid (which includes
// the cells next to flavour thresholds).
//
// Training is deterministic: every reduction has a fixed order (within a
// 64-row slice of the batch, then the slices in order), so a checkpointed and
// resumed run reproduces a straight run bit for bit.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "interp_dev.h"
#include "pdfmi_dev.h"

namespace pdfmi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kH = 64;   // hidden width
constexpr int kO = 16;   // output width (stored columns padded)
// flat FP32 parameter layout
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kH * 2, kOffW2 = kOffB1 + kH, kOffB2 = kOffW2 + kH * kH,
              kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH * kH, kOffW4 = kOffB3 + kH, kOffB4 = kOffW4 + kO * kH,
              kNParams = kOffB4 + kO;
// BF16 parameter block (SurBufs::Pb): [0, n) hi halves, [n, 2n) lo halves in
// the flat layout, then the hi halves of W2, W3 and W4 transposed (the
// backward pass multiplies with them; kept transposed by whatever writes the
// parameters, so that a training step stages them with plain 16-byte copies).
constexpr int kOffW2t = 2 * kNParams, kOffW3t = kOffW2t + kH * kH, kOffW4t = kOffW3t + kH * kH,
              kNPb = kOffW4t + kH * kO;
static_assert(kOffW2 % 8 == 0 && kOffW3 % 8 == 0 && kOffW4 % 8 == 0 && kNParams % 8 == 0, "16-byte staging copies");

__device__ __forceinline__ unsigned short bf16_bits(float f) {
  const __bf16 h = (__bf16)f;  // round to nearest even
  return __builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ float bf16_float(unsigned short b) {
  return __uint_as_float(((unsigned)b) << 16);
}
// BF16 pair of v: hi = bf16(v), lo = bf16(v - hi) (the difference is exact in FP32)
__device__ __forceinline__ void split_bits(float v, unsigned short& hi, unsigned short& lo) {
  hi = bf16_bits(v);
  lo = bf16_bits(v - bf16_float(hi));
}

// BF16 halves of parameter i into the block Pb, and its transposed hi half.
__device__ __forceinline__ void store_halves(unsigned short* __restrict__ Pb, int i, float p) {
  unsigned short hi, lo;
  split_bits(p, hi, lo);
  Pb[i] = hi;
  Pb[kNParams + i] = lo;
  if (i >= kOffW2 && i < kOffB2) Pb[kOffW2t + ((i - kOffW2) % kH) * kH + (i - kOffW2) / kH] = hi;
  if (i >= kOffW3 && i < kOffB3) Pb[kOffW3t + ((i - kOffW3) % kH) * kH + (i - kOffW3) / kH] = hi;
  if (i >= kOffW4 && i < kOffB4) Pb[kOffW4t + ((i - kOffW4) % kH) * kO + (i - kOffW4) / kH] = hi;
}

// tanh(z) = 1 - 2 / (exp(2z) + 1) from the hardware exp2 and reciprocal:
// exp2 overflows to +inf (result 1) and underflows to 0 (result -1); near 0
// the absolute error is a few 1e-8, far below the BF16 rounding of the
// activations.
constexpr float kTwoLog2e = 2.8853900817779268f;  // 2 log2(e)
// tanh(z) from zs = 2 log2(e) z (inference folds the factor into its weights and biases)
__device__ __forceinline__ float tanh_scaled(float zs) {
  return fmaf(-2.0f, __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(zs) + 1.0f), 1.0f);
}
__device__ __forceinline__ float tanh_f(float z) { return tanh_scaled(kTwoLog2e * z); }

// ---------------------------------------------------------------------------------------
// Training step, fused into two launches.  k_train_fb: one workgroup of 16
// waves per 64-row slice of the batch runs the forward and backward passes
// (wave (row group, t) owns rows R0 .. R0 + 15 and units 16 t .. 16 t + 15 of
// every hidden layer; activations stay in registers and LDS) and writes the
// slice's gradient and its sum of squared errors to the workspace.  What
// bounds it is the chain of six layers, each a few dependent LDS reads,
// MFMAs, tanh and a barrier: with four waves of 16 rows x 64 units each SIMD
// held one wave and waited out every latency (10.8 us a launch at batch 4096;
// 8.8 us with four waves per SIMD; 14.7 us when the transposed weights were
// also formed here, two bytes at a time, and biases and targets were loaded
// where they are used).  One extra workgroup computes the step's
// learning rate and bias corrections (FP64 powers and a cosine) beside the
// others.  k_train_update (k_grad_reduce without the update) adds the slices
// in slice order and applies Adam.
//
// Matrix products on v_mfma_f32_16x16x32_bf16: lane l = 16 g + r holds
// A(row r, k = 8 g .. 8 g + 7) and B(k = 8 g .. 8 g + 7, column r) of a
// 32-deep step and receives C(rows 4 g .. 4 g + 3, column r).  The forward
// products take the three split terms per k step (hi*hi, lo*hi, hi*lo) and
// walk k in order; the backward products multiply BF16 (hi) signals with the
// hi halves.  Weight gradients sum over the slice's 64 rows in two k steps,
// bias gradients (and the FP32 first-layer weight gradient) over each lane's
// four rows, then lanes g = 0..3 of row groups 0..3 in that order.
//
// LDS tiles of BF16 with 64 columns are rows of 128 bytes whose 16-byte
// chunks are rotated by (row & 7), so that the 16-byte operand reads of eight
// lanes on consecutive rows hit eight different chunk positions; tiles of 16
// columns (32-byte rows) swap their two chunks on rows 4..7 of every eight.
constexpr int kTRows = 64, kTGroups = kTRows / 16, kTThreads = 64 * kTGroups * 4;
constexpr int kNPad = (kNParams + 1 + 63) / 64 * 64;  // workspace stride per slice: gradient, then the loss sum

__device__ __forceinline__ int swz64(int row, int col) {
  return row * 128 + ((((col >> 3) ^ row) & 7) << 4) + ((col & 7) << 1);
}
__device__ __forceinline__ int swz16(int row, int col) {
  return row * 32 + ((((col >> 3) ^ (row >> 2)) & 1) << 4) + ((col & 7) << 1);
}
__device__ __forceinline__ bf16x8 ld8(const unsigned char* base, int off) {
  return *reinterpret_cast<const bf16x8*>(base + off);
}
__device__ __forceinline__ void st_bf16(unsigned char* base, int off, unsigned short v) {
  *reinterpret_cast<unsigned short*>(base + off) = v;
}
// four consecutive columns c .. c + 3 (c a multiple of 4) of one row
__device__ __forceinline__ void st4_bf16(unsigned char* base, int off, const unsigned short v[4]) {
  *reinterpret_cast<uint2*>(base + off) =
      make_uint2((unsigned)v[0] | ((unsigned)v[1] << 16), (unsigned)v[2] | ((unsigned)v[3] << 16));
}

// Byte offsets of the LDS regions of k_train_fb.
constexpr int kT64 = 64 * 64 * 2, kT16 = 64 * 16 * 2;
constexpr int kLW2h = 0, kLW2l = kLW2h + kT64, kLW3h = kLW2l + kT64, kLW3l = kLW3h + kT64;  // W[n][k]
constexpr int kLW2t = kLW3l + kT64, kLW3t = kLW2t + kT64;                                   // W^T[k][n], hi
constexpr int kLW4h = kLW3t + kT64, kLW4l = kLW4h + kT16, kLW4t = kLW4l + kT16;           // W4[o][k]; W4^T[k][o]
constexpr int kLAh0 = kLW4t + kT16, kLAl0 = kLAh0 + kT64, kLAh1 = kLAl0 + kT64, kLAl1 = kLAh1 + kT64;  // layer inputs
constexpr int kLH1t = kLAl1 + kT64, kLH2t = kLH1t + kT64, kLH3t = kLH2t + kT64;  // activations^T [unit][row], hi
constexpr int kLDz = kLH3t + kT64, kLDzt = kLDz + kT64;                          // dz [row][unit], dz^T, hi
constexpr int kLDy = kLDzt + kT64, kLDyt = kLDy + kT16;                          // dy [row][o], dy^T [o][row]
constexpr int kLIn = kLDyt + kT16;                                               // in [row][2], FP32
constexpr int kLRed = kLIn + kTRows * 2 * 4;                                     // [3][waves][4][64] FP32
constexpr int kLLoss = kLRed + 3 * kTGroups * 4 * 64 * 4;                        // [row groups] FP32
constexpr int kTrainLds = kLLoss + kTGroups * 4;

// The three split products of one 32-deep k step, in the order hi*hi, lo*hi, hi*lo.
__device__ __forceinline__ f32x4 mfma3(bf16x8 a, bf16x8 al, bf16x8 b, bf16x8 bl, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, c, 0, 0, 0);
}

// Stores a hidden layer's outputs h (this lane's rows 4 g + i, column 16 t + r)
// as the next layer's split A operand and as hi^T for the weight gradient.
__device__ __forceinline__ void store_hidden(unsigned char* L, int ah, int al, int ht, int R0, int t, int g, int r,
                                             const float h[4]) {
  unsigned short hi[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    split_bits(h[i], hi[i], lo[i]);
    st_bf16(L + ah, swz64(R0 + 4 * g + i, 16 * t + r), hi[i]);
    st_bf16(L + al, swz64(R0 + 4 * g + i, 16 * t + r), lo[i]);
  }
  st4_bf16(L + ht, swz64(16 * t + r, R0 + 4 * g), hi);
}

// Hidden layer 2 or 3 forward: h = tanh(A W^T + b) for this wave's rows and units.
__device__ __forceinline__ void hidden_fwd(const unsigned char* L, int ah, int al, int wh, int wl, float bias,
                                           int R0, int t, int g, int r, float h[4]) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k0 = 0; k0 < kH; k0 += 32)
    acc = mfma3(ld8(L + ah, swz64(R0 + r, k0 + 8 * g)), ld8(L + al, swz64(R0 + r, k0 + 8 * g)),
                ld8(L + wh, swz64(16 * t + r, k0 + 8 * g)), ld8(L + wl, swz64(16 * t + r, k0 + 8 * g)), acc);
#pragma unroll
  for (int i = 0; i < 4; ++i) h[i] = tanh_f(acc[i] + bias);
}

// 16 x 16 tile (output units R0 .., input units 16 t ..) of a 64-unit layer's
// weight gradient: dW[j][i] = sum over the slice's rows of dz[b][j] h[b][i] (hi operands).
__device__ __forceinline__ void weight_grad(const unsigned char* L, int dzt, int ht, int R0, int t, int g, int r,
                                            float* __restrict__ out) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k0 = 0; k0 < kTRows; k0 += 32)
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(L + dzt, swz64(R0 + r, k0 + 8 * g)),
                                                  ld8(L + ht, swz64(16 * t + r, k0 + 8 * g)), acc, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) out[(R0 + 4 * g + i) * kH + 16 * t + r] = acc[i];
}

// dh = dz W for this wave's rows and units (K = the 64 output units, W^T staged).
__device__ __forceinline__ f32x4 input_grad(const unsigned char* L, int dz, int wt, int R0, int t, int g, int r) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k0 = 0; k0 < kH; k0 += 32)
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(L + dz, swz64(R0 + r, k0 + 8 * g)),
                                                  ld8(L + wt, swz64(16 * t + r, k0 + 8 * g)), acc, 0, 0, 0);
  return acc;
}

// dz = dh (1 - h^2) (tanh derivative): its hi halves to the dz and dz^T
// tiles; this lane's sum over its four rows to red[row group][g].
__device__ __forceinline__ void tanh_back(unsigned char* L, float* red, const float h[4], f32x4 dh, int R0, int t,
                                          int g, int r) {
  unsigned short hi[4];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float dz = dh[i] * (1.0f - h[i] * h[i]);
    hi[i] = bf16_bits(dz);
    st_bf16(L + kLDz, swz64(R0 + 4 * g + i, 16 * t + r), hi[i]);
    s += dz;
  }
  st4_bf16(L + kLDzt, swz64(16 * t + r, R0 + 4 * g), hi);
  red[((R0 >> 4) * 4 + g) * 64 + 16 * t + r] = s;
}

// Column c's sum of red[row group w][g][c] over w = 0..3, g = 0..3 in that order.
__device__ __forceinline__ float red_sum(const float* red, int c) {
  float s = red[c];
#pragma unroll
  for (int q = 1; q < kTGroups * 4; ++q) s += red[q * 64 + c];
  return s;
}

// Learning rate and bias corrections of update number st->step + 1, into st:
// cosine schedule lrf + (lr0 - lrf)(1 + cos(pi min(1, step / total))) / 2; the
// betas' powers in FP64, as the host computes them.
__device__ void schedule(SurStep* st) {
  const double t = (double)st->step;
  const double frac = fmin(1.0, t / (double)st->total);
  st->lr = (float)(st->lrf + 0.5 * ((double)st->lr0 - st->lrf) * (1.0 + cos(3.141592653589793 * frac)));
  st->c1 = (float)(1.0 - pow(0.9, t + 1.0));
  st->c2 = (float)(1.0 - pow(0.999, t + 1.0));
}

__global__ __launch_bounds__(kTThreads) void k_train_fb(const float* __restrict__ in, const float* __restrict__ T,
                                                        SurStep* __restrict__ st, const float* __restrict__ P,
                                                        const unsigned short* __restrict__ Pb, int B,
                                                        float* __restrict__ ws) {
  if (st && blockIdx.x == gridDim.x - 1) {  // the extra workgroup of a training step (see above)
    if (threadIdx.x == 0) schedule(st);
    return;
  }
  extern __shared__ __align__(16) unsigned char L[];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 15, g = lane >> 4;
  const int R0 = 16 * (w & 3), t = w >> 2, u = 16 * t + r;  // rows R0 .., this lane's unit
  const int64_t row0 = (st ? st->row : 0) + (int64_t)blockIdx.x * kTRows;
  const int nrow = min(kTRows, B - (int)blockIdx.x * kTRows);  // valid rows of this slice
  float* out = ws + (int64_t)blockIdx.x * kNPad;
  float* red = reinterpret_cast<float*>(L + kLRed);

  // this lane's biases, first-layer weights and targets (registers), and the
  // weights on their way to LDS: split W2, W3, W4 row-major; hi of W2^T, W3^T,
  // W4^T.  Every global load of the step is issued before the first wait.
  const float w10 = P[kOffW1 + 2 * u], w11 = P[kOffW1 + 2 * u + 1], b1 = P[kOffB1 + u], b2 = P[kOffB2 + u],
              b3 = P[kOffB3 + u], b4 = P[kOffB4 + r];
  float tr[4];
  {
    auto src = [](const unsigned short* base, int c) { return *reinterpret_cast<const uint4*>(base + 8 * c); };
    // 16-byte chunk c of a 64 x 64 matrix (row c / 8, columns 8 (c % 8) ..); threads 0..511 take
    // the hi, lo and transposed copies of W2, the others those of W3
    const int c = tid & 511;
    const bool two = tid < 512;
    const uint4 qh = src(Pb + (two ? kOffW2 : kOffW3), c);
    const uint4 ql = src(Pb + kNParams + (two ? kOffW2 : kOffW3), c);
    const uint4 qt = src(Pb + (two ? kOffW2t : kOffW3t), c);
    // W4 (16 rows of 8 chunks): hi by threads 0..127, lo by 128..255; W4^T (64 rows of 2) by 256..383
    const int c4 = tid & 127, part = tid >> 7;
    uint4 q4 = make_uint4(0, 0, 0, 0);
    if (part < 3) q4 = src(Pb + (part == 0 ? kOffW4 : (part == 1 ? kNParams + kOffW4 : kOffW4t)), c4);
    float xin = 0.0f;
    if (part == 3 && c4 < 2 * nrow) xin = in[2 * row0 + c4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = R0 + 4 * g + i;
      tr[i] = t == 0 && b < nrow ? T[(row0 + b) * kO + r] : 0.0f;
    }
    const int d = swz64(c >> 3, (c & 7) * 8);
    *reinterpret_cast<uint4*>(L + (two ? kLW2h : kLW3h) + d) = qh;
    *reinterpret_cast<uint4*>(L + (two ? kLW2l : kLW3l) + d) = ql;
    *reinterpret_cast<uint4*>(L + (two ? kLW2t : kLW3t) + d) = qt;
    if (part < 2) *reinterpret_cast<uint4*>(L + (part == 0 ? kLW4h : kLW4l) + swz64(c4 >> 3, (c4 & 7) * 8)) = q4;
    if (part == 2) *reinterpret_cast<uint4*>(L + kLW4t + swz16(c4 >> 1, (c4 & 1) * 8)) = q4;
    if (part == 3) reinterpret_cast<float*>(L + kLIn)[c4] = xin;
  }
  __syncthreads();
  const float* sin = reinterpret_cast<const float*>(L + kLIn);

  // layer 1 (FP32): h1[b][u] = tanh(W1[u][0] in[b][0] + W1[u][1] in[b][1] + b1[u])
  float h1[4], h2[4], h3[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = R0 + 4 * g + i;
    h1[i] = tanh_f(fmaf(w10, sin[2 * b], fmaf(w11, sin[2 * b + 1], b1)));
  }
  store_hidden(L, kLAh0, kLAl0, kLH1t, R0, t, g, r, h1);
  __syncthreads();
  hidden_fwd(L, kLAh0, kLAl0, kLW2h, kLW2l, b2, R0, t, g, r, h2);
  store_hidden(L, kLAh1, kLAl1, kLH2t, R0, t, g, r, h2);
  __syncthreads();
  hidden_fwd(L, kLAh1, kLAl1, kLW3h, kLW3l, b3, R0, t, g, r, h3);
  store_hidden(L, kLAh0, kLAl0, kLH3t, R0, t, g, r, h3);
  __syncthreads();

  // layer 4 and the loss (one wave per row group): y = h3 W4^T + b4; d = y - T; dy = 2 d / (B kO)
  if (t == 0) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < kH; k0 += 32)
      acc = mfma3(ld8(L + kLAh0, swz64(R0 + r, k0 + 8 * g)), ld8(L + kLAl0, swz64(R0 + r, k0 + 8 * g)),
                  ld8(L + kLW4h, swz64(r, k0 + 8 * g)), ld8(L + kLW4l, swz64(r, k0 + 8 * g)), acc);
    const float scale = (float)((int64_t)B * kO);
    unsigned short hi[4];
    float sq = 0.0f, s = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = R0 + 4 * g + i;
      const float d = b < nrow ? (acc[i] + b4) - tr[i] : 0.0f;
      const float gr = 2.0f * d / scale;
      hi[i] = bf16_bits(gr);
      st_bf16(L + kLDy, swz16(b, r), hi[i]);
      sq += d * d;
      s += gr;
    }
    st4_bf16(L + kLDyt, swz64(r, R0 + 4 * g), hi);
    red[(w * 4 + g) * 64 + r] = s;
    // the wave's sum of squares, pairs of lanes first (a fixed order)
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) sq += __shfl_xor(sq, m);
    if (lane == 0) reinterpret_cast<float*>(L + kLLoss)[w] = sq;
  }
  __syncthreads();

  // layer 4 backward: dh3 = dy W4; dW4 (wave of row group w: input units 16 w ..), db4, the loss
  const bf16x8 zero = {};
  f32x4 dh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g < 2 ? ld8(L + kLDy, swz16(R0 + r, 8 * g)) : zero,  // K = 16 of 32
                                                     g < 2 ? ld8(L + kLW4t, swz16(u, 8 * g)) : zero,
                                                     f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  if (t == 1) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < kTRows; k0 += 32)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(L + kLDyt, swz64(r, k0 + 8 * g)),
                                                    ld8(L + kLH3t, swz64(R0 + r, k0 + 8 * g)), acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[kOffW4 + (4 * g + i) * kH + R0 + r] = acc[i];
  }
  if (tid < kO) out[kOffB4 + tid] = red_sum(red, tid);
  if (tid == 64) {
    const float* ls = reinterpret_cast<const float*>(L + kLLoss);
    out[kNParams] = ((ls[0] + ls[1]) + ls[2]) + ls[3];
  }
  __syncthreads();  // red and the loss sums consumed

  // layer 3 backward
  tanh_back(L, red, h3, dh, R0, t, g, r);
  __syncthreads();
  dh = input_grad(L, kLDz, kLW3t, R0, t, g, r);
  weight_grad(L, kLDzt, kLH2t, R0, t, g, r, out + kOffW3);
  if (tid < kH) out[kOffB3 + tid] = red_sum(red, tid);
  __syncthreads();
  // layer 2 backward
  tanh_back(L, red, h2, dh, R0, t, g, r);
  __syncthreads();
  dh = input_grad(L, kLDz, kLW2t, R0, t, g, r);
  weight_grad(L, kLDzt, kLH1t, R0, t, g, r, out + kOffW2);
  if (tid < kH) out[kOffB2 + tid] = red_sum(red, tid);
  __syncthreads();
  // layer 1 backward (FP32): dW1[u][k] = sum_b dz[b][u] in[b][k], db1
  float s0 = 0.0f, s1 = 0.0f, sb = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = R0 + 4 * g + i;
    const float dz = dh[i] * (1.0f - h1[i] * h1[i]);
    s0 = fmaf(dz, sin[2 * b], s0);
    s1 = fmaf(dz, sin[2 * b + 1], s1);
    sb += dz;
  }
  const int q = ((w & 3) * 4 + g) * 64 + u;
  red[q] = s0;
  red[kTGroups * 4 * 64 + q] = s1;
  red[2 * kTGroups * 4 * 64 + q] = sb;
  __syncthreads();
  if (tid < 3 * kH) {  // one wave each for the two weight columns and the bias
    const float v = red_sum(red + w * kTGroups * 4 * 64, lane);
    out[w < 2 ? kOffW1 + 2 * lane + w : kOffB1 + lane] = v;
  }
}

// Adam step of parameter i (Kingma & Ba, bias-corrected moments; c1 = 1 -
// b1^t, c2 = 1 - b2^t for update number t), then its BF16 pair.
__device__ __forceinline__ void adam_update(int i, float g, float lr, float b1, float b2, float eps, float c1,
                                            float c2, float* __restrict__ P, float* __restrict__ Mm,
                                            float* __restrict__ Vm, unsigned short* __restrict__ Pb) {
  const float m = b1 * Mm[i] + (1.0f - b1) * g;
  const float v = b2 * Vm[i] + (1.0f - b2) * g * g;
  Mm[i] = m;
  Vm[i] = v;
  const float p = P[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  P[i] = p;
  store_halves(Pb, i, p);
}

// Adam with a given gradient G (pdf_surrogate_adam).
__global__ void k_adam(float* __restrict__ P, const float* __restrict__ G, float* __restrict__ Mm,
                       float* __restrict__ Vm, unsigned short* __restrict__ Pb, int n, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam_update(i, G[i], lr, b1, b2, eps, c1, c2, P, Mm, Vm, Pb);
}

// Gradient i = sum over the S slices of the workspace, in slice order.  The
// loads of kSliceLoads slices are in flight at a time: one after another they
// cost a memory latency each (64 slices: k_train_update took 30.7 us, now 5.5).
constexpr int kSliceLoads = 32;
__device__ __forceinline__ float slice_sum(const float* __restrict__ ws, int S, int i) {
  float g = 0.0f;
  for (int q0 = 0; q0 < S; q0 += kSliceLoads) {
    float v[kSliceLoads];
#pragma unroll
    for (int q = 0; q < kSliceLoads; ++q) v[q] = ws[(int64_t)min(q0 + q, S - 1) * kNPad + i];
#pragma unroll
    for (int q = 0; q < kSliceLoads; ++q)
      if (q0 + q < S) g = q0 + q == 0 ? v[0] : g + v[q];
  }
  return g;
}

// The gradient and loss of k_train_fb's slices (no update).
__global__ __launch_bounds__(256) void k_grad_reduce(const float* __restrict__ ws, int S, float* __restrict__ G,
                                                     float inv_n, float* __restrict__ loss,
                                                     float* __restrict__ loss_out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kNParams) G[i] = slice_sum(ws, S, i);
  if (i == 0) {
    const float l = slice_sum(ws, S, kNParams) * inv_n;
    *loss = l;
    if (loss_out) *loss_out = l;
  }
}

// Gradient of the slices and Adam at the step's learning rate (computed by
// k_train_fb), one thread per parameter; one further thread forms the loss
// and advances the step state, which no other thread of this kernel reads.
// Workgroups of one wave spread the 2.4 MB of partial gradients over 150 CUs.
constexpr int kUpdThreads = 64;
__global__ __launch_bounds__(kUpdThreads) void k_train_update(const float* __restrict__ ws, int S,
                                                              float* __restrict__ P, float* __restrict__ G,
                                                              float* __restrict__ Mm, float* __restrict__ Vm,
                                                              unsigned short* __restrict__ Pb, float inv_n,
                                                              float* __restrict__ loss, int B,
                                                              SurStep* __restrict__ st) {
  const int i = blockIdx.x * kUpdThreads + threadIdx.x;
  if (i < kNParams) {
    const float lr = st->lr, c1 = st->c1, c2 = st->c2;
    const float g = slice_sum(ws, S, i);
    G[i] = g;
    adam_update(i, g, lr, 0.9f, 0.999f, 1e-8f, c1, c2, P, Mm, Vm, Pb);
  } else if (i == kNParams) {
    const float l = slice_sum(ws, S, kNParams) * inv_n;
    *loss = l;
    if (st->loss_out) st->loss_out[st->call] = l;
    st->step += 1;
    st->row = (st->step % st->nb) * (int64_t)B;
    st->call += 1;
  }
}

// Start of a training call: the global step, the call's step index, the schedule and the loss output.
__global__ void k_train_begin(SurStep* st, int64_t step, int64_t nb, int B, int total, float lr0, float lrf,
                              float* loss_out) {
  st->step = step;
  st->call = 0;
  st->nb = nb;
  st->row = (step % nb) * (int64_t)B;
  st->total = total;
  st->lr0 = lr0;
  st->lrf = lrf;
  st->loss_out = loss_out;
}

__global__ void k_to_bf16(const float* __restrict__ P, unsigned short* __restrict__ Pb, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) store_halves(Pb, i, P[i]);
}

// ---------------------------------------------------------------------------------------
// Envelope and sample preparation.

// Hermite weights of the envelope at ln x: cell i (largest i <= nx-2 with
// lxk[i] <= ln x, clamped) and the basis h00, h10 D, h01, h11 D of its
// parameter t (clamped to [0, 1]), D = lxk[i+1] - lxk[i].
struct EnvW {
  int i;
  float h00, h10, h01, h11;
};

// Weights of cell i, of width D, at cell parameter u.
__device__ __forceinline__ EnvW env_cell(int i, double u, double D) {
  const double t = fmin(fmax(u, 0.0), 1.0);
  const double s = 1.0 - t, t2 = t * t, s2 = s * s;  // factored basis: no cancellation near t = 0, 1
  EnvW w;
  w.i = i;
  w.h00 = (float)(s2 * (1.0 + 2.0 * t));
  w.h10 = (float)(t * s2 * D);
  w.h01 = (float)(t2 * (3.0 - 2.0 * t));
  w.h11 = (float)(-(s * t2) * D);
  return w;
}

__device__ __forceinline__ EnvW env_weights(const double* lxk, int nx, double lx) {
  int lo = 0, hi = nx - 2;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (lxk[mid] <= lx) lo = mid; else hi = mid - 1;
  }
  const double D = lxk[lo + 1] - lxk[lo];
  return env_cell(lo, (lx - lxk[lo]) / D, D);
}

// E_c at the point whose weights are w (tables [nx][kO] of values and slopes)
__device__ __forceinline__ float env_at(const float* e, const float* d, int i, float h00, float h10, float h01,
                                        float h11, int c) {
  const int a = i * kO + c, b = a + kO;
  return fmaf(h00, e[a], fmaf(h10, d[a], fmaf(h01, e[b], h11 * d[b])));
}

// Columns c .. c + 3 (c a multiple of 4), by 16-byte reads.
__device__ __forceinline__ f32x4 env_at4(const float* e, const float* d, int i, f32x4 h, int c) {
  const int a = i * kO + c;
  const f32x4 e0 = *reinterpret_cast<const f32x4*>(e + a), d0 = *reinterpret_cast<const f32x4*>(d + a);
  const f32x4 e1 = *reinterpret_cast<const f32x4*>(e + a + kO), d1 = *reinterpret_cast<const f32x4*>(d + a + kO);
  f32x4 r;
#pragma unroll
  for (int q = 0; q < 4; ++q) r[q] = fmaf(h[0], e0[q], fmaf(h[1], d0[q], fmaf(h[2], e1[q], h[3] * d1[q])));
  return r;
}

__device__ __forceinline__ bool trusted(const SurDev& S, const MemberDev& m, double x, double q2) {
  if (!(x >= m.xmin && x <= m.xmax && q2 >= m.qmin && q2 <= m.qmax)) return false;
  int k = 0;
  for (int j = 1; j < S.K; ++j)
    if (S.qfirst[j] <= q2) k = j;
  return S.trust[k] && x >= S.txlo[k] && x < S.txhi[k] && q2 >= S.tqlo[k] && q2 < S.tqhi[k];
}

// Normalised inputs, targets xf_c / E_c (0 where E_c = 0 or xf is not
// finite) and whether the sample lies in the network's domain.
__global__ void k_prep_samples(SurDev S, MemberDev m, const double* __restrict__ X, const double* __restrict__ Q2,
                               const double* __restrict__ XF, int64_t n, float* __restrict__ in,
                               float* __restrict__ T, unsigned char* __restrict__ keep) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = X[i], q2 = Q2[i];
  keep[i] = trusted(S, m, x, q2) ? 1 : 0;
  const double lx = log(x), lq = log(q2);
  in[2 * i] = (float)(2.0 * (lx - S.lx0) * S.ilx - 1.0);
  in[2 * i + 1] = (float)(2.0 * (lq - S.lq0) * S.ilq - 1.0);
  const EnvW w = env_weights(S.lxk, S.nx, lx);
  for (int c = 0; c < kO; ++c) {
    float t = 0.0f;
    if (c < S.P) {
      const float e = env_at(S.env, S.envd, w.i, w.h00, w.h10, w.h01, w.h11, c);
      const double xf = XF[i * S.P + c];
      if (e != 0.0f && isfinite(xf)) t = (float)(xf / (double)e);
    }
    T[i * kO + c] = t;
  }
}

// in[j], T[j] = in_all[idx[j]], T_all[idx[j]] for j < n (the kept samples, in order).
__global__ void k_gather_samples(const float* __restrict__ in_all, const float* __restrict__ T_all,
                                 const int64_t* __restrict__ idx, int64_t n, float* __restrict__ in,
                                 float* __restrict__ T) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int64_t i = idx[j];
  in[2 * j] = in_all[2 * i];
  in[2 * j + 1] = in_all[2 * i + 1];
#pragma unroll
  for (int c = 0; c < kO; ++c) T[j * kO + c] = T_all[i * kO + c];
}

// ---------------------------------------------------------------------------------------
// Fused inference.  Each wave takes 64 consecutive points: their inputs,
// fallback flags and envelope weights are prepared one lane per point (cell
// and logarithms from the member's location tables), then the network runs on
// two sub-tiles of 32 points with the activations kept in registers from
// layer to layer.  Each layer is formed transposed on the matrix cores,
// h' = tanh(W h + b) with the weights as the A operand and two columns of 16
// points' activations as B operands, three products per operand pair: lane
// (r, g) then receives units 16 t + 4 g + i (t, i = 0..3) of point r, which
// are the 16 values it supplies to the next layer's B operand when that
// layer's 64-deep k index k' = 32 s + 8 g + i stands for unit
// kunit(k') = 16 (2 s + i / 4) + 4 g + i % 4.  The weight columns are staged
// in LDS in that order (once per workgroup), so no activation passes through
// LDS.  Layer 1 is one FP32 matrix product per 16 units, of (W1, b1) with
// (u, v, 1), with the argument scale of tanh_scaled folded in.  In layers 2
// and 3 only the biases carry that scale: folded into the weights before
// their split it saves one instruction per activation (3.5 % of the time), but
// scaled weights use their BF16 binades differently, and the error against an
// FP64 network grew from 3.80e-6 to 3.98e-6 (relative rms, 400 networks of
// uniform weights).  The outputs
// times the envelope go to a 32 x 16 LDS tile from which the requested
// columns are stored point-major, consecutive lanes on consecutive values,
// by a walk that is laid out once per workgroup.  Points in the fallback
// domain are queued per wave and evaluated 64 at a time by the FP32
// interpolator over what the network wrote: each is located once (one lane
// per point: sub-grid, cells, weights), after which one lane per (point,
// requested column) gathers its 4x4 stencil.
//
// What bounds it is the vector work of the activations: 192 per point, each
// an exp2 and a reciprocal at half rate and six more instructions.  10^7
// points of 11 columns: 1215 us with 16-point sub-tiles, layer 1 and the bias
// on the vector units, the halves split by unpacking and two library FP64
// logarithms and a binary search per point; 1027 us with each weight fragment
// read for 32 points, layer 1 on the matrix cores and the table lookups; about
// 950 us with the split by dot products and the output walk; 915 us with
// 16-byte staging, all tables in flight together.
//
// LDS rows of 64 BF16 values (the weight halves) hold their eight 16-byte
// chunks in the order chunk ^ (row & 7), so the 16 rows an operand read
// touches spread over the banks.  Blocks of 16 waves fill the CU's LDS
// (4 waves per SIMD, at most 128 VGPRs; 12 waves without register spills
// measured 936 us against 908).
constexpr int kSurWaves = 16;
constexpr int kSurPts = 32;  // points of a sub-tile: two MFMA columns of 16
// Tiles go to the workgroups first and to their waves second, and calls of up
// to this many 32-point tiles per compute unit take tiles of 32: a wave alone
// needs about 3 us per 32 points, sixteen on one compute unit 24.  (16 tiles of
// 64 points to each workgroup in turn: 1000 points on one compute unit, 32.3
// us a call, now 12.2; 10^5 34.5 -> 22.5; 3 10^5 58 -> 38.5.  With 64-point
// tiles 1000 points take 17 us; from 10^5 points on it makes no difference.)
constexpr int kSurSmallWaves = 8;
constexpr int kSurRec = 8;   // floats per point record: u, v, h00, h10 D, h01, h11 D, cell, (unused)

__device__ __forceinline__ int swz(int row, int col) {  // element offset of (row, col) in a swizzled [.][64] tile
  return row * kH + ((((col >> 3) ^ row) & 7) << 3) + (col & 7);
}
// Hidden unit that the k index k' of a layer's B operand stands for (see above).
__device__ __forceinline__ int kunit(int kp) {
  return ((kp >> 5) << 5) + (((kp >> 2) & 1) << 4) + (((kp >> 3) & 3) << 2) + (kp & 3);
}

// Four activations tanh from their scaled arguments, split, into values o .. o + 3 of an operand.
__device__ __forceinline__ void act4(f32x4 z, bf16x8& hi, bf16x8& lo, int o, bf16x2 m0, bf16x2 m1) {
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const float v0 = tanh_scaled(z[i]), v1 = tanh_scaled(z[i + 1]);
    const bf16x2 h = {(__bf16)v0, (__bf16)v1};
    hi[o + i] = h[0];
    hi[o + i + 1] = h[1];
    // v - hi (exact) as a dot product with (-1, 0) or (0, -1): no unpacking of the two halves
    lo[o + i] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(h, m0, v0, false);
    lo[o + i + 1] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(h, m1, v1, false);
  }
}

// Location of one fallback point.
// Rows here are whole 16-byte units, so the low four bits of the record's s1
// and s3 are free: they hold the mode of a point outside the grid.
struct FbRec {
  PointRec<float> r;
  double p0, p1;  // extrapolation parameters
};
__device__ __forceinline__ void fb_set_mode(FbRec& f, int mode) {
  f.r.s1 |= mode & 15;  // region
  f.r.s3 |= (mode & kXHigh ? 1 : 0) | ((mode >> 8) & 3) << 1;
}
__device__ __forceinline__ float fb_extrapolate(const FbRec& f, const float* col0, int Pp, double invL01,
                                                const LogEntry* lt) {
  const int mode = (f.r.s1 & 15) | (f.r.s3 & 1 ? kXHigh : 0) | ((f.r.s3 >> 1) & 3) << 8;
  PointRec<float> r = f.r;
  r.s1 &= ~15;
  r.s3 &= ~15;
  return rec_extrapolate<float, true>(r, mode, f.p0, f.p1, col0, Pp, invL01, lt);
}

// LDS of k_sur_infer: the lo and hi halves of W2, W3 (64 x 64) and W4
// (16 x 64) with their columns in kunit order, [nx] ln x knots (double),
// [nx][16] envelope values and slopes, b2 and b3 times 2 log2(e) (the
// argument scale of tanh_scaled), b4, the output walk; then
// per wave a 5 KB area (4 KB for the output tile, later the fallback records;
// 1 KB for the fallback queue) and the point records.
constexpr size_t kSurWaveArea = 4096 + 128 * 8;  // output tile or fallback records, then the fallback queue
constexpr size_t kSurWTile = (size_t)2 * (2 * kH * kH + kO * kH);  // one half of W2, W3, W4 (BF16)
__host__ __device__ static inline size_t sur_head_bytes(int nx) {
  const size_t b = 2 * kSurWTile + (size_t)8 * (nx + (nx & 1)) +
                   (size_t)4 * (2 * nx * kO + 2 * kH + kO + kMaxReq) + (size_t)2 * kSurPts * kMaxReq;
  return (b + 15) & ~(size_t)15;
}
constexpr size_t kSurWaveBytes = kSurWaveArea + 64 * kSurRec * 4;
// Waves per block: kSurWaves, fewer when the per-block tables (which grow
// with the number of x knots) leave less LDS.
int sur_infer_waves(int nx) {
  const size_t head = sur_head_bytes(nx);
  const size_t lds = 160 * 1024;
  const int w = head >= lds ? 0 : (int)((lds - head) / kSurWaveBytes);
  return w < kSurWaves ? w : kSurWaves;
}
size_t sur_infer_shared_bytes(int nx, int waves) { return sur_head_bytes(nx) + (size_t)waves * kSurWaveBytes; }

__global__ __launch_bounds__(64 * kSurWaves) __attribute__((amdgpu_waves_per_eu(4)))
void k_sur_infer(SurDev S, MemberDev m, ReqCols rc, const float* __restrict__ Pf,
                 const double* __restrict__ X, const double* __restrict__ Q2, int64_t n, float* __restrict__ out, double invL01, unsigned long long* __restrict__ nerr, int tile_pts) {
  extern __shared__ __align__(16) unsigned char sraw[];
  const int BS = blockDim.x, nwav = BS >> 6;
  unsigned short* sw2l = reinterpret_cast<unsigned short*>(sraw);  // [kH][kH] swizzled (16-byte chunks)
  unsigned short* sw3l = sw2l + kH * kH;
  unsigned short* sw4l = sw3l + kH * kH;                   // [kO][kH] swizzled
  unsigned short* sw2h = sw4l + kO * kH;                   // hi halves, same layout
  unsigned short* sw3h = sw2h + kH * kH;
  unsigned short* sw4h = sw3h + kH * kH;
  double* slxk = reinterpret_cast<double*>(sw4h + kO * kH);  // [nx]
  float* senv = reinterpret_cast<float*>(slxk + S.nx + (S.nx & 1));  // [nx][kO], 16-byte aligned
  float* senvd = senv + S.nx * kO;                         // [nx][kO]
  float* sb2 = senvd + S.nx * kO;
  float* sb3 = sb2 + kH;
  float* sb4 = sb3 + kH;                                   // [kO]
  int* scol = reinterpret_cast<int*>(sb4 + kO);            // [kMaxReq] stored column of each requested flavour
  unsigned short* swalk = reinterpret_cast<unsigned short*>(scol + kMaxReq);  // [kSurPts][R] offset in the output tile
  unsigned char* waves = sraw + sur_head_bytes(S.nx);
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, r = l & 15, g = l >> 4;
  unsigned char* area = waves + (size_t)wv * kSurWaveArea;
  float* so = reinterpret_cast<float*>(area);                         // [kSurPts][kO] output tile
  FbRec* fbr = reinterpret_cast<FbRec*>(area);                        // [64] fallback records
  int64_t* fq = reinterpret_cast<int64_t*>(area + 4096);              // [128] queued fallback points
  static_assert(64 * sizeof(FbRec) <= 4096, "fallback records fit the wave area");
  float* rec = reinterpret_cast<float*>(waves + (size_t)nwav * kSurWaveArea) + wv * 64 * kSurRec;

  // staging, 16 bytes a load and the first of every table in flight together
  // (four stored columns kp .. kp + 3 of row n hold W[n][kunit(kp)] and the
  // three units after it)
  const f32x4* e4 = reinterpret_cast<const f32x4*>(S.env);
  const f32x4* d4 = reinterpret_cast<const f32x4*>(S.envd);
  const int ne4 = S.nx * kO / 4;
  auto unit4 = [&](int off, int i) {  // chunk i of the matrix at off, in stored order
    return *reinterpret_cast<const f32x4*>(Pf + off + (i / (kH / 4)) * kH + kunit(4 * (i % (kH / 4))));
  };
  auto stage4 = [&](f32x4 w, unsigned short* hi, unsigned short* lo, int i) {
    bf16x4 h, l4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      h[q] = (__bf16)w[q];
      l4[q] = (__bf16)(w[q] - (float)h[q]);
    }
    const int o = swz(i / (kH / 4), 4 * (i % (kH / 4)));
    *reinterpret_cast<bf16x4*>(hi + o) = h;
    *reinterpret_cast<bf16x4*>(lo + o) = l4;
  };
  {
    const int i = threadIdx.x;
    const f32x4 e = e4[min(i, ne4 - 1)], d = d4[min(i, ne4 - 1)];
    const f32x4 w2 = unit4(kOffW2, i), w3 = unit4(kOffW3, i), w4 = unit4(kOffW4, i & (kO * kH / 4 - 1));
    const float c2 = Pf[kOffB2 + (i & (kH - 1))], c3 = Pf[kOffB3 + (i & (kH - 1))], c4 = Pf[kOffB4 + (i & (kO - 1))];
    const double lk = S.lxk[min(i, S.nx - 1)];
    stage4(w2, sw2h, sw2l, i);
    stage4(w3, sw3h, sw3l, i);
    if (i < kO * kH / 4) stage4(w4, sw4h, sw4l, i);
    if (i < ne4) {
      reinterpret_cast<f32x4*>(senv)[i] = e;
      reinterpret_cast<f32x4*>(senvd)[i] = d;
    }
    if (i < kH) {
      sb2[i] = kTwoLog2e * c2;
      sb3[i] = kTwoLog2e * c3;
    }
    if (i < kO) sb4[i] = c4;
    if (i < S.nx) slxk[i] = lk;
  }
  for (int i = threadIdx.x + BS; i < kH * kH / 4; i += BS) {
    stage4(unit4(kOffW2, i), sw2h, sw2l, i);
    stage4(unit4(kOffW3, i), sw3h, sw3l, i);
    if (i < kO * kH / 4) stage4(unit4(kOffW4, i), sw4h, sw4l, i);
  }
  for (int i = threadIdx.x + BS; i < ne4; i += BS) {
    reinterpret_cast<f32x4*>(senv)[i] = e4[i];
    reinterpret_cast<f32x4*>(senvd)[i] = d4[i];
  }
  for (int i = threadIdx.x + BS; i < S.nx; i += BS) slxk[i] = S.lxk[i];
  for (int i = threadIdx.x; i < rc.n; i += BS) scol[i] = rc.col[i];
  for (int i = threadIdx.x; i < kSurPts * rc.n; i += BS) {
    const int pt = i / rc.n, c = rc.col[i - pt * rc.n];
    swalk[i] = (unsigned short)(c < 0 ? 0xffff : pt * kO + c);
  }
  __syncthreads();

  // layer 1 as the FP32 product [W1 | b1 | 0] (u, v, 1, 0): this lane's A operand, row 16 t + r, k = g
  float w1[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int j = 16 * t + r;
    w1[t] = g == 3 ? 0.0f : kTwoLog2e * Pf[g == 2 ? kOffB1 + j : kOffW1 + 2 * j + g];
  }

  unsigned mb0 = 0x0000bf80u, mb1 = 0xbf800000u;  // BF16 (-1, 0) and (0, -1), in registers
  asm("" : "+s"(mb0), "+s"(mb1));
  const bf16x2 m0 = __builtin_bit_cast(bf16x2, mb0), m1 = __builtin_bit_cast(bf16x2, mb1);
  // an 8-value chunk (16 bytes) of a swizzled LDS row, as an operand fragment
  auto frag = [&](const unsigned short* tile, int row, int col0) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(tile + swz(row, col0));
  };
  const Tables gtb = tables_at(m.tables, m);
  const float* __restrict__ gvals = member_values<float>(m);
  const int R = rc.n;

  const int64_t ntiles = (n + tile_pts - 1) / tile_pts;
  int qn = 0;  // queued fallback points of this wave (fewer than 64 between tiles)
  for (int64_t tile = (int64_t)wv * gridDim.x + blockIdx.x; tile < ntiles; tile += (int64_t)gridDim.x * nwav) {
    const int64_t p0 = tile * tile_pts;
    const int np = (int)min((int64_t)tile_pts, n - p0);
    // one lane per point: inputs, fallback flag, envelope weights
    double xr = 0.5, qr = 1.0;
    bool fb = false;
    float* pr = rec + l * kSurRec;
    if (l < np) {
      xr = X[p0 + l];
      qr = Q2[p0 + l];
      fb = !trusted(S, m, xr, qr);
      // x cell and ln x from the member's location tables (any x gives a cell in range)
      const int ei = find_cell(gtb.knots + m.xk_off, m.nx, xr, m.xh, gtb.hints);
      const CellCoef& c = entry<CellCoef>(gtb.cells, m.xc_off + ei);
      const double l = fast_log(xr * c.inv_t0, gtb.logt);
      pr[0] = (float)(2.0 * (slxk[ei] + l - S.lx0) * S.ilx - 1.0);
      pr[1] = (float)(2.0 * (fast_log(qr, gtb.logt) - S.lq0) * S.ilq - 1.0);
      const EnvW ew = env_cell(ei, l * c.invD, slxk[ei + 1] - slxk[ei]);
      pr[2] = ew.h00;
      pr[3] = ew.h10;
      pr[4] = ew.h01;
      pr[5] = ew.h11;
      pr[6] = __int_as_float(ew.i);
    } else {
      pr[0] = pr[1] = pr[2] = pr[3] = pr[4] = pr[5] = 0.0f;
      pr[6] = __int_as_float(0);
    }
    const unsigned long long fbmask = __ballot(fb);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int q0 = 0; q0 < np; q0 += kSurPts) {
      // B operands (hi, lo) of the two columns of 16 points: bh[p][s][i] is unit kunit(32 s + 8 g + i) of
      // point q0 + 16 p + r
      bf16x8 bh[2][2], bl[2][2];
      // layer 1: lane (k = g, column r) supplies u, v, 1, 0 and receives units 16 t + 4 g + i of point r
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const float in = g < 2 ? rec[(q0 + 16 * p + r) * kSurRec + g] : (g == 2 ? 1.0f : 0.0f);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const f32x4 z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[2 * s + t], in, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            act4(z, bh[p][s], bl[p][s], 4 * t, m0, m1);
          }
      }
      // layers 2 and 3: each weight fragment read once for both columns
#pragma unroll
      for (int layer = 0; layer < 2; ++layer) {
        const float* bias = layer == 0 ? sb2 : sb3;
        const unsigned short* wh = layer == 0 ? sw2h : sw3h;
        const unsigned short* wl = layer == 0 ? sw2l : sw3l;
        bf16x8 nh[2][2], nl[2][2];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + 16 * t + 4 * g);
          f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const bf16x8 ah = frag(wh, 16 * t + r, 32 * s + 8 * g), al = frag(wl, 16 * t + r, 32 * s + 8 * g);
#pragma unroll
            for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[p][s], acc[p], 0, 0, 0);
#pragma unroll
            for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[p][s], acc[p], 0, 0, 0);
#pragma unroll
            for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[p][s], acc[p], 0, 0, 0);
          }
#pragma unroll
          for (int p = 0; p < 2; ++p) act4(acc[p] * kTwoLog2e + bv, nh[p][t >> 1], nl[p][t >> 1], 4 * (t & 1), m0, m1);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            bh[p][s] = nh[p][s];
            bl[p][s] = nl[p][s];
          }
      }
      // layer 4: lane (r, g) gets y[output 4 g + i][point]; times the envelope into the output tile
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(sb4 + 4 * g);
      f32x4 y[2] = {b4, b4};
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf16x8 ah = frag(sw4h, r, 32 * s + 8 * g), al = frag(sw4l, r, 32 * s + 8 * g);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          y[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[p][s], y[p], 0, 0, 0);
          y[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[p][s], y[p], 0, 0, 0);
          y[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[p][s], y[p], 0, 0, 0);
        }
      }
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const float* pq = rec + (q0 + 16 * p + r) * kSurRec;
        const f32x4 hw = {pq[2], pq[3], pq[4], pq[5]};
        *reinterpret_cast<f32x4*>(so + (16 * p + r) * kO + 4 * g) =
            y[p] * env_at4(senv, senvd, __float_as_int(pq[6]), hw, 4 * g);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // requested columns, point-major: consecutive lanes on consecutive values (a fallback point's are
      // written over below, by this wave)
      const int ne = min(kSurPts, np - q0) * R;
      float* o = out + (p0 + q0) * R;
      for (int e = l; e < ne; e += 64) {
        const int w = swalk[e];
        o[e] = w != 0xffff ? so[w] : 0.0f;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // fallback points: queued, and evaluated 64 at a time (one lane per point
    // locates it, then one lane per (point, requested column) gathers), so the
    // location runs on full waves rather than on the few fallback lanes of
    // every tile
    if (fb) fq[qn + __popcll(fbmask & ((1ull << l) - 1))] = p0 + l;
    qn += __popcll(fbmask);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool last = tile + (int64_t)gridDim.x * nwav >= ntiles;
    while (qn >= 64 || (last && qn > 0)) {
      const int nfb = min(qn, 64);
      bool bad = false;
      if (l < nfb) {
        FbRec& fr = fbr[l];
        const int64_t pi = fq[l];
        const double xf = X[pi], qf = Q2[pi];
        const QLoc<float> Q = locate_q<float>(m, gtb, qf);
        const PointLoc L = locate_x<float>(m, gtb, Q, xf, qf, fr.r.w, fr.r.v);
        set_stencil(fr.r, Q, L, m.P32 * 4);
        fb_set_mode(fr, L.mode);
        fr.p0 = L.p0;
        fr.p1 = L.p1;
        bad = L.mode & kInvalid;
      }
      const unsigned long long badm = __ballot(bad);
      if (badm && l == 0) atomicAdd(nerr, (unsigned long long)__popcll(badm));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (int e = l; e < nfb * R; e += 64) {
        const int k = e / R, j = e - k * R;
        const FbRec& fr = fbr[k];
        const int c = scol[j];
        float val;
        if (fr.r.o & kRecInvalid) {
          val = NAN;
        } else if (c < 0) {
          val = 0.0f;
        } else if (!(fr.r.o & kRecSlow)) {
          const float* f0 = gvals + c + fr.r.o / 4;
          const int s1 = fr.r.s1 / 4, sa = fr.r.sa / 4, s3 = fr.r.s3 / 4;
          const float* fx[4] = {f0, f0 + s1, f0 + s1 + sa, f0 + s1 + sa + s3};
          float F[4][4];
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) F[a][b] = fx[a][b * m.P32];
          val = interp_stencil<float>(F, fr.r.w, fr.r.v);
        } else {
          val = fb_extrapolate(fr, gvals + c, m.P32, invL01, gtb.logt);
        }
        out[fq[k] * R + j] = val;
      }
      // the rest of the queue (fewer than 64) to its front: the two ranges do not overlap
      const int rest = qn - nfb;
      const int64_t mv = l < rest ? fq[nfb + l] : 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (l < rest) fq[l] = mv;
      qn = rest;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

}  // namespace pdfmi

namespace pdfmi {

// ---------------------------------------------------------------------------------------
// Host-side launchers.


int sur_nparams() { return kNParams; }
int sur_halves() { return kNPb; }
int sur_out_width() { return kO; }
int sur_hidden() { return kH; }

static unsigned nb(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Slices of a batch of B rows in the fused training step, and the workspace
// (floats) their partial gradients and losses take.
int sur_slices(int B) { return (B + kTRows - 1) / kTRows; }
size_t sur_workspace_floats(int B) { return (size_t)sur_slices(B) * kNPad; }

// LDS limit of the fused step; called before a step is first launched or recorded.
hipError_t sur_train_prepare() {
  return allow_dynamic_lds(reinterpret_cast<const void*>(&k_train_fb), kTrainLds);
}

// One forward + backward pass on a batch (inputs in[B][2], targets T[B][kO])
// with no update: gradient into buf.G, loss (mean squared error) into
// buf.loss and, if not null, *loss_out.
hipError_t sur_forward_backward(const SurBufs& b, const float* in, const float* T, int B, float* loss_out,
                                hipStream_t s) {
  hipError_t e = sur_train_prepare();
  if (e != hipSuccess) return e;
  const int S = sur_slices(B);
  hipLaunchKernelGGL(k_train_fb, dim3((unsigned)S), dim3(kTThreads), kTrainLds, s, in, T, (SurStep*)nullptr,
                     b.P, b.Pb, B, b.wpart);
  hipLaunchKernelGGL(k_grad_reduce, dim3(nb(kNParams, 256)), dim3(256), 0, s, b.wpart, S, b.G,
                     1.0f / (float)((int64_t)B * kO), b.loss, loss_out);
  return hipGetLastError();
}

hipError_t sur_adam(const SurBufs& b, float lr, int step, hipStream_t s) {
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - pow(b1, step)), c2 = (float)(1.0 - pow(b2, step));
  hipLaunchKernelGGL(k_adam, dim3(nb(kNParams, 256)), dim3(256), 0, s, b.P, b.G, b.M, b.V, b.Pb, kNParams, lr,
                     (float)b1, (float)b2, 1e-8f, c1, c2);
  return hipGetLastError();
}

// Start of a training call (the state the step kernels read).
hipError_t sur_train_begin(const SurBufs& b, int64_t step, int64_t nbatches, int B, int total, float lr0, float lrf,
                           float* loss_out, hipStream_t s) {
  hipLaunchKernelGGL(k_train_begin, dim3(1), dim3(1), 0, s, b.st, step, nbatches, B, total, lr0, lrf, loss_out);
  return hipGetLastError();
}

// One training step on the slice of the training set (in, T) that b.st
// selects: the fused forward + backward pass, then the slice sums, Adam at
// the scheduled learning rate and the step advance.  The same two launches
// at every step (recorded once as a graph by the caller); sur_train_prepare
// must have run.
hipError_t sur_train_step(const SurBufs& b, const float* in, const float* T, int B, hipStream_t s) {
  const int S = sur_slices(B);
  hipLaunchKernelGGL(k_train_fb, dim3((unsigned)S + 1), dim3(kTThreads), kTrainLds, s, in, T, b.st, b.P, b.Pb, B,
                     b.wpart);
  hipLaunchKernelGGL(k_train_update, dim3(nb(kNParams + 1, kUpdThreads)), dim3(kUpdThreads), 0, s, b.wpart, S, b.P,
                     b.G, b.M, b.V, b.Pb, 1.0f / (float)((int64_t)B * kO), b.loss, B, b.st);
  return hipGetLastError();
}

hipError_t sur_refresh_bf16(const SurBufs& b, hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3(nb(kNParams, 256)), dim3(256), 0, s, b.P, b.Pb, kNParams);
  return hipGetLastError();
}

hipError_t sur_prep(const SurDev& S, const MemberDev& m, const double* x, const double* q2, const double* xf,
                    int64_t n, float* in, float* T, unsigned char* keep, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_prep_samples, dim3(nb(n, 256)), dim3(256), 0, s, S, m, x, q2, xf, n, in, T, keep);
  return hipGetLastError();
}

hipError_t sur_gather(const float* in_all, const float* T_all, const int64_t* idx, int64_t n, float* in, float* T,
                      hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_gather_samples, dim3(nb(n, 256)), dim3(256), 0, s, in_all, T_all, idx, n, in, T);
  return hipGetLastError();
}

hipError_t sur_infer(const SurDev& S, const MemberDev& m, const ReqCols& rc, const SurBufs& b, const double* x,
                     const double* q2, int64_t n, float* out, double invL01, unsigned long long* nerr, int n_cu,
                     hipStream_t s) {
  const int waves = sur_infer_waves(S.nx);
  if (waves < 1) return hipErrorInvalidValue;  // envelope tables beyond LDS (the create call bounds nx)
  const size_t shm = sur_infer_shared_bytes(S.nx, waves);
  const int64_t per_cu = std::max<int64_t>(1, (int64_t)(160 * 1024) / (int64_t)shm);
  const int tile_pts = n <= (int64_t)n_cu * kSurSmallWaves * kSurPts ? kSurPts : 64;
  const int64_t tiles = (n + tile_pts - 1) / tile_pts;
  const int64_t blocks = min(tiles, (int64_t)n_cu * per_cu);
  if (blocks > 0) {
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&k_sur_infer), shm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sur_infer, dim3((unsigned)blocks), dim3(64 * waves), shm, s, S, m, rc, b.P, x, q2, n,
                       out, invL01, nerr, tile_pts);
  }
  return hipGetLastError();
}

}  // namespace pdfmi
