// Learned right-hand-side correction: a 108 -> 256 -> 256 -> 12 GELU network
// in BF16 with FP32 accumulation on the gfx950 matrix cores (v_mfma 16x16x32
// bf16), its backward pass and Adam, the 3x3-stencil features of an r = 1
// state, and the learned stage (plain r = 1 right-hand side + correction, with
// a per-element trust bound and a global mass correction).
//
// MFMA 16x16x32 bf16 operand layout (lane l of 64): A[row = l%16][k = 8(l/16)+j],
// B[k = 8(l/16)+j][col = l%16], j = 0..7; result C[row = 4(l/16)+i][col = l%16],
// i = 0..3.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dgsw_ctx.hpp"
#include "dgsw_device.hpp"
#include "dgsw_mlp.hpp"

namespace dgsw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// GELU(z) = z Phi(z) = (z/2)(1 + erf(z / sqrt 2)) with erf from the rational
// approximation of Abramowitz & Stegun, formula 7.1.26 (Hastings): for x >= 0,
// erf(x) = 1 - P(t) exp(-x^2), t = 1 / (1 + p x),
// P(t) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))), absolute error <= 1.5e-7,
// far below the BF16 rounding the activations then take.  Since erf is odd,
// z erf(z / sqrt 2) = |z| (1 - P exp(-z^2 / 2)), so
//   GELU(z)  = max(z, 0) - |z| P / 2 exp(-z^2 / 2),
//   GELU'(z) = Phi(z) + z phi(z) = [z >= 0] - sgn(z) P / 2 e + z e / sqrt(2 pi),
// e = exp(-z^2 / 2): branch-free, one hardware reciprocal and one hardware
// base-2 exponential each.  The A&S coefficients enter halved (P / 2) and p
// is scaled by 1 / sqrt 2 (t from |z| directly).
namespace gelu_as {
constexpr float kP = 0.3275911f * 0.70710678118654752f;
constexpr float kA1 = 0.5f * 0.254829592f, kA2 = 0.5f * -0.284496736f, kA3 = 0.5f * 1.421413741f,
                kA4 = 0.5f * -1.453152027f, kA5 = 0.5f * 1.061405429f;
constexpr float kHalfLog2e = 0.72134752044448170f;   // log2(e) / 2: exp(-z^2/2) = 2^(-z^2 log2(e)/2)
__device__ __forceinline__ float half_poly(float az) {
  const float t = __builtin_amdgcn_rcpf(fmaf(kP, az, 1.0f));
  return t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, kA5, kA4), kA3), kA2), kA1);
}
__device__ __forceinline__ float gauss(float z) { return __builtin_amdgcn_exp2f(-(z * z) * kHalfLog2e); }
}  // namespace gelu_as

__device__ __forceinline__ float gelu_f(float z) {
  const float az = fabsf(z);
  // max(z, 0) on the bits: fmaxf() also quiets its operand, one more
  // instruction of 15 (a NaN reaches the sum through az)
  const float zp = __int_as_float(max(__float_as_int(z), 0));
  return fmaf(-az * gelu_as::half_poly(az), gelu_as::gauss(z), zp);
}
// GELU(z) and, in place of z, GELU'(z): one reciprocal and one exponential for both.
__device__ __forceinline__ float gelu_and_grad(float &z) {
  const float az = fabsf(z), hp = gelu_as::half_poly(az), e = gelu_as::gauss(z);
  const float h = fmaf(-az * hp, e, fmaxf(z, 0.0f));
  z = fmaf(e, fmaf(z, 0.39894228040143268f, -copysignf(hp, z)), z >= 0.0f ? 1.0f : 0.0f);
  return h;
}

// ------------------------------------------------------------------ fused inference
// The whole network in one persistent kernel: one workgroup of 8 wavefronts
// per compute unit, looping over tiles of 64 rows.  Each wavefront loads its
// slice of the two hidden layers' weights into registers once (32 units of
// each, from the fragment order of k_prep_weights: one contiguous kilobyte
// per load) and keeps them for every tile, the output layer's weights are
// copied to LDS, so the weights cross the cache hierarchy once per workgroup
// instead of once per 64 rows.  Per tile the BF16 inputs
// (stencil features computed from an r = 1 state, or given FP32 rows) and
// both hidden layers stay in LDS; only the inputs and the FP32 outputs touch
// global memory.  Each product is computed transposed, out^T = W in^T: the
// weights are the MFMA A operand (row = unit, 8 consecutive k per lane) and
// the LDS rows the B operand, so every lane ends with 4 consecutive units of
// one row and writes them as one 8-byte LDS store.  Rounding points: BF16
// inputs, weights and hidden activations, FP32 accumulation, bias and GELU in
// FP32.  By its counters the vector unit is busy 0.47 of the time (most of it the
// GELU, 14 instructions per unit and row), the matrix cores 0.14, and 0.30 of the
// wavefronts' time waits for memory or a barrier.  Inputs have a buffer of their
// own, so a tile has three barriers and the next tile's operands are fetched
// meanwhile: with the operands fetched at the tile's start and rows padded instead
// of permuted 40.0 us for 64 800 rows, now 35.6 (36.8 before the weights were
// requested behind the first tile's inputs); weights streamed from L2 for two
// workgroups per CU took 38.8.
constexpr int kRows = 64;                 // rows per tile
constexpr int kMlpGrid = 256;             // persistent workgroups: one per MI355X compute unit
template <typename T>
struct MlpCorrection {           // the learned stage's correction step (FROM_Q)
  const T *L1;
  const float *omean, *ostd;
  const double *mass_w;
  float kappa;
  float *C;
  double *partial;
  int64_t *fallback;
};
constexpr int kWaves = 8;                 // wavefronts per workgroup
constexpr int kLd = kHidden + 8;          // LDS row stride in BF16 (+16 B: no bank conflicts)
constexpr int kYs = kRows + 4;            // stride of the network outputs' unit columns in LDS
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Offset in BF16 of the 16-byte chunk c of an LDS row of whole 256-byte
// multiples: chunks are permuted within a row by the row's index, so that the
// rows a wavefront reads or writes at one column lie in different banks
// whatever 16 lanes the unit takes together.  (Rows padded by 16 bytes
// instead: half of the cycles of the reads were bank conflicts.)
__device__ __forceinline__ int swz(int c, int row) { return (c ^ (row & 15)) * 8; }

// One hidden layer for the 64 rows of a tile: wavefront wv computes units
// [32 wv, 32 wv + 32) of out = gelu(in W^T + b), K inputs per row, from the
// weight fragments w[ks][nt] it holds.
template <int K>
__device__ __forceinline__ void fused_hidden(const bf16x8 (&w)[K / 32][2], const float *bias, const __bf16 *in,
                                             __bf16 *out, int wv, int lane) {
  constexpr int NT = 2, MT = kRows / 16, KS = K / 32;
  const int r = lane & 15, kc = lane >> 4;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + 32 * wv + 16 * nt + kc * 4);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = bv;   // the bias, then the products
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    bf16x8 b[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      b[mt] = *reinterpret_cast<const bf16x8 *>(in + (16 * mt + r) * K + swz(4 * ks + kc, r));
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt], b[mt], acc[nt][mt], 0, 0, 0);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int col = swz(4 * wv + 2 * nt + (kc >> 1), r) + 4 * (kc & 1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = (__bf16)gelu_f(acc[nt][mt][i]);
      *reinterpret_cast<bf16x4 *>(out + (16 * mt + r) * kHidden + col) = h;
    }
  }
}

// This wavefront's weight fragments of a hidden layer (units 32 wv ..), from
// the fragment order Wf (one contiguous kilobyte per load), and the matching
// biases.
template <int K>
__device__ __forceinline__ void load_hidden(const __bf16 *__restrict__ Wf, int wv,
                                            int lane, bf16x8 (&w)[K / 32][2]) {
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const __bf16 *blk = Wf + (size_t)(2 * wv + nt) * (K / 32) * 512 + lane * 8;
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks) w[ks][nt] = *reinterpret_cast<const bf16x8 *>(blk + 512 * ks);
  }
}

// Per-element correction from the network output y[12] (standardised), as
// k_correction: c = mean_j + std_j y with c_(h,00) = 0; rejected (c = 0) if
// non-finite or, for a variable, max|c| > kappa max|L1|.  Returns whether it
// fell back and the element's h-mass of the correction.
template <int SY, int SL>
__device__ __forceinline__ bool correction_row(const float *y, const float *L1e, const float *om, const float *os,
                                               float kappa, float *c) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    c[k] = k == 0 ? 0.f : om[k * SL] + os[k * SL] * y[k * SY];
    ok = ok && isfinite(c[k]);
  }
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    float mc = 0.f, ml = 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      mc = fmaxf(mc, fabsf(c[v * 4 + m]));
      ml = fmaxf(ml, fabsf(L1e[(v * 4 + m) * SL]));
    }
    ok = ok && !(mc > kappa * ml);
  }
  if (!ok) {
#pragma unroll
    for (int k = 0; k < 12; ++k) c[k] = 0.f;
  }
  return !ok;
}

// FROM_Q: features of the r = 1 state q (as k_features), then the correction
// of every element (the learned stage): C[rows][12], the workgroup's h-mass
// of the corrections (summed over its tiles in tile order) in
// partial[blockIdx.x] and the fallback count; else the network on rows of
// X[rows][108], output Y[rows][32].  Tiles blockIdx.x, blockIdx.x + gridDim.x, ..
template <typename T, bool FROM_Q>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(64 * kWaves) void k_mlp_fused(const T *__restrict__ q, int n_lon, int n_lat,
                                                          const float *__restrict__ fmean,
                                                          const float *__restrict__ fistd,
                                                          const float *__restrict__ X, int rows,
                                                          const __bf16 *__restrict__ W1f,
                                                          const __bf16 *__restrict__ W2f,
                                                          const __bf16 *__restrict__ W3t,
                                                          const float *__restrict__ b1, const float *__restrict__ b2,
                                                          const float *__restrict__ b3p, float *__restrict__ Y,
                                                          MlpCorrection<T> cor) {
  __shared__ __attribute__((aligned(16))) __bf16 bufx[kRows * kInPad];    // inputs
  __shared__ __attribute__((aligned(16))) __bf16 buf1[kRows * kHidden];   // first and second hidden layer
  __shared__ __attribute__((aligned(16))) __bf16 buf2[kRows * kHidden];
  __shared__ __attribute__((aligned(16))) __bf16 st_w3[kOutPad * kHidden];
  __shared__ __attribute__((aligned(16))) float st_b1[kHidden], st_b2[kHidden];
  __shared__ float ys[FROM_Q ? kOutPad * kYs : 1];                        // outputs, for the correction
  // the correction's operands of the tile's rows (FROM_Q): the r = 1
  // right-hand side, the output mean and spread of the row's latitude (value
  // k of row i at k kRows + i: the lane-per-row reads hit distinct banks), the
  // latitude's h-mass weight of mode (0, 1)
  __shared__ float st_l1[FROM_Q ? kRows * 12 : 1], st_om[FROM_Q ? kRows * 12 : 1], st_os[FROM_Q ? kRows * 12 : 1];
  __shared__ double st_mw[FROM_Q ? kRows : 1];
  // the feature standardisation (FROM_Q), once per workgroup
  __shared__ float st_fm[FROM_Q ? kFeatures : 1], st_fi[FROM_Q ? kFeatures : 1];
  int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // output layer: wavefront wv takes rows [16 (wv / 2), +16) and units [16 (wv % 2), +16)
  const int mt = wv >> 1, nt = wv & 1;
  double mass = 0.0;          // wavefront 0: this workgroup's h-mass of the corrections
  bool any_fell = false;
  unsigned long long fell_count = 0ull;
  // Input tasks, one per (row, stencil neighbour) of a tile: 12 contiguous
  // values, and their BF16 features in bufx.
  using In = typename std::conditional<FROM_Q, T, float>::type;
  auto task_src = [&](int e0, int task) -> const In * {
    const int rr = task / 9, sn = task - rr * 9;
    const int e = e0 + rr < rows ? e0 + rr : rows - 1;
    if constexpr (FROM_Q) {
      const int dj = sn / 3 - 1, di = sn % 3 - 1;
      const int j = e / n_lon, i = e - j * n_lon;
      int jj = j + dj;
      jj = jj < 0 ? 0 : (jj >= n_lat ? n_lat - 1 : jj);
      int ii = i + di;
      ii = ii < 0 ? ii + n_lon : (ii >= n_lon ? ii - n_lon : ii);
      return q + ((size_t)jj * n_lon + ii) * 12;
    } else {
      return X + (size_t)e * kFeatures + sn * 12;
    }
  };
  auto store_task = [&](int task, auto value) {
    const int rr = task / 9, sn = task - rr * 9;
    float x[12];
#pragma unroll
    for (int vm = 0; vm < 12; ++vm) x[vm] = value(vm);
    if constexpr (FROM_Q) {
#pragma unroll
      for (int vm = 0; vm < 12; ++vm) x[vm] = (x[vm] - st_fm[sn * 12 + vm]) * st_fi[sn * 12 + vm];
    }
#pragma unroll
    for (int h4 = 0; h4 < 3; ++h4)
      *reinterpret_cast<bf16x4 *>(bufx + rr * kInPad + swz((3 * sn + h4) >> 1, rr) + 4 * ((3 * sn + h4) & 1)) =
          bf16x4{(__bf16)x[4 * h4], (__bf16)x[4 * h4 + 1], (__bf16)x[4 * h4 + 2], (__bf16)x[4 * h4 + 3]};
  };
  // The operands of a tile that come from memory, requested before its first
  // layer and stored after a later one: raw, the next tile's input tasks;
  // half, per lane two pieces of 6 In each: wavefront kExtra the tasks beyond
  // one per lane, wavefronts 1 .. 3 the correction's operands of this tile's
  // rows (the right-hand side, then the output mean and spread, 12 floats each:
  // with FP64 one piece, with FP32 two); wavefront 5 the h-mass weight.
  constexpr int kTasks = kRows * 9, kExtra = 4;
  static_assert(kTasks > 64 * kWaves && kTasks <= 64 * kWaves + 64, "one extra task per lane of one wavefront");
  constexpr bool kWide = sizeof(In) == 8;
  constexpr int kWords = 3 * sizeof(In);            // of the 12 values, in 32 bits
  In raw[12];
  unsigned half[kWords];
  double mw = 0.0;
  auto load_tile = [&](int e0, int e0n) {
    const In *src = task_src(e0n, tid);
#pragma unroll
    for (int vm = 0; vm < 12; ++vm) raw[vm] = src[vm];
    if (FROM_Q ? (wv >= 1 && wv <= kExtra) : wv == kExtra) {
      const In *p0 = nullptr, *p1 = nullptr;
      if (wv == kExtra) {
        p0 = task_src(e0n, lane + 64 * kWaves);
        p1 = p0 + 6;
      } else if constexpr (FROM_Q) {
        const int e = e0 + lane < rows ? e0 + lane : rows - 1;
        const int j = e / n_lon;
        if (wv == 1) {
          p0 = cor.L1 + (size_t)e * 12;
          p1 = p0 + 6;
        } else {
          const float *f0 = (wv == 2 ? cor.omean : cor.ostd) + j * 12;
          p0 = reinterpret_cast<const In *>(f0);
          p1 = kWide ? reinterpret_cast<const In *>(cor.ostd + j * 12) : p0 + 6;
        }
      }
      const unsigned *u0 = reinterpret_cast<const unsigned *>(p0), *u1 = reinterpret_cast<const unsigned *>(p1);
#pragma unroll
      for (int k = 0; k < kWords / 2; ++k) half[k] = u0[k];
#pragma unroll
      for (int k = 0; k < kWords / 2; ++k) half[kWords / 2 + k] = u1[k];
    }
    if constexpr (FROM_Q) {
      if (wv == 5) {
        const int e = e0 + lane < rows ? e0 + lane : rows - 1;
        mw = cor.mass_w[e / n_lon * 2 + 1];
      }
    }
  };
  auto half_value = [&](int k) -> float {
    if constexpr (kWide)
      return (float)__hiloint2double((int)half[2 * k + 1], (int)half[2 * k]);
    else
      return __uint_as_float(half[k]);
  };
  auto store_operands = [&]() {
    if (wv == 1) {
#pragma unroll
      for (int k = 0; k < 12; ++k) st_l1[k * kRows + lane] = half_value(k);
    } else if (wv == 2 || (!kWide && wv == 3)) {
      float *dst = (wv == 2 ? st_om : st_os) + lane;
#pragma unroll
      for (int k = 0; k < 12; ++k) dst[k * kRows] = __uint_as_float(half[k]);
      if constexpr (kWide) {
#pragma unroll
        for (int k = 0; k < 12; ++k) st_os[k * kRows + lane] = __uint_as_float(half[12 + k]);
      }
    } else if (wv == 5) {
      st_mw[lane] = mw;
    }
  };
  auto store_inputs = [&]() {
    store_task(tid, [&](int k) { return (float)raw[k]; });
    if (wv == kExtra) store_task(lane + 64 * kWaves, half_value);
  };
  const int ntiles = (rows + kRows - 1) / kRows;
  load_tile(blockIdx.x * kRows, blockIdx.x * kRows);
  // the tables in LDS, all loads issued before any is waited for: the output
  // layer's weights (chunks permuted like the activations; registers held for
  // 8 products per tile would push the kernel into scratch), the biases, the
  // feature standardisation
  constexpr int kChunks = kOutPad * kHidden / 8 / (64 * kWaves);
  static_assert(kOutPad * kHidden == 8 * 64 * kWaves * kChunks && 2 * kHidden == 64 * kWaves && kFeatures <= 64 * kWaves,
                "table copies");
  bf16x8 w3c[kChunks];
#pragma unroll
  for (int n = 0; n < kChunks; ++n) w3c[n] = *reinterpret_cast<const bf16x8 *>(W3t + 8 * (tid + 64 * kWaves * n));
  const float bias = tid < kHidden ? b1[tid] : b2[tid - kHidden];
  const int kf = tid < kFeatures ? tid : 0;
  const float fm = FROM_Q ? fmean[kf] : 0.f, fi = FROM_Q ? fistd[kf] : 0.f;
  const f32x4 bv3 = *reinterpret_cast<const f32x4 *>(b3p + 16 * nt + (lane >> 4) * 4);
  // the hidden layers' weights in registers, requested after the first tile's
  // operands and the LDS tables (loads complete in order: the tables and the
  // inputs wait only for their own, and the second layer's weights arrive
  // during the first layer)
  bf16x8 w1[kInPad / 32][2], w2[kHidden / 32][2];
  load_hidden<kInPad>(W1f, wv, lane, w1);
  load_hidden<kHidden>(W2f, wv, lane, w2);
#pragma unroll
  for (int n = 0; n < kChunks; ++n) {
    const int c = tid + 64 * kWaves * n, u = c / (kHidden / 8), k8 = c - u * (kHidden / 8);
    *reinterpret_cast<bf16x8 *>(st_w3 + u * kHidden + swz(k8, u)) = w3c[n];
  }
  if (tid < kHidden)
    st_b1[tid] = bias;
  else
    st_b2[tid - kHidden] = bias;
  if (FROM_Q && tid < kFeatures) {
    st_fm[tid] = fm;
    st_fi[tid] = fi;
  }
  // zero padding of the inputs beyond the 108 features (never overwritten)
  for (int idx = tid; idx < kRows * (kInPad - kFeatures) / 4; idx += 64 * kWaves) {
    const int rr = idx / ((kInPad - kFeatures) / 4), k = kFeatures + 4 * (idx - rr * ((kInPad - kFeatures) / 4));
    *reinterpret_cast<bf16x4 *>(bufx + rr * kInPad + swz(k >> 3, rr) + (k & 4)) = bf16x4{};
  }
  __syncthreads();            // the tables above before their first use
  store_inputs();
  __syncthreads();
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int e0 = tile * kRows;
    // opaque to the compiler: offsets that depend on the lane alone are formed
    // again for each tile, not held in registers beside the weights
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    const int r = lane & 15, kc = lane >> 4, n0 = 16 * nt + 4 * kc;
    load_tile(e0, tile + (int)gridDim.x < ntiles ? (tile + (int)gridDim.x) * kRows : e0);   // (after the last: not used)
    fused_hidden<kInPad>(w1, st_b1, bufx, buf1, wv, lane);
    __syncthreads();   // and wavefront 0 has left the last tile's correction
    if constexpr (FROM_Q) store_operands();
    fused_hidden<kHidden>(w2, st_b2, buf1, buf2, wv, lane);
    store_inputs();    // every wavefront has left the first layer
    __syncthreads();
    f32x4 acc = bv3;
    bf16x8 b[kHidden / 32], w3[kHidden / 32];
#pragma unroll
    for (int ks = 0; ks < kHidden / 32; ++ks) {
      b[ks] = *reinterpret_cast<const bf16x8 *>(buf2 + (16 * mt + r) * kHidden + swz(4 * ks + kc, r));
      w3[ks] = *reinterpret_cast<const bf16x8 *>(st_w3 + (16 * nt + r) * kHidden + swz(4 * ks + kc, r));
    }
#pragma unroll
    for (int ks = 0; ks < kHidden / 32; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3[ks], b[ks], acc, 0, 0, 0);
    const f32x4 out = acc;
    if constexpr (!FROM_Q) {
      const int e = e0 + 16 * mt + r;
      if (e < rows) *reinterpret_cast<f32x4 *>(Y + (size_t)e * kOutPad + n0) = out;
    } else {
      // outputs to LDS, then one lane per row forms its element's correction
      // (wavefront 0, while the others go on to the next tile's first layer)
      // (unit n of row i at n kYs + i: conflict-free stores and lane-per-row reads)
#pragma unroll
      for (int i = 0; i < 4; ++i) ys[(n0 + i) * kYs + 16 * mt + r] = out[i];
      __syncthreads();
      if (wv == 0) {
        const int e = e0 + lane;
        double m = 0.0;
        bool fell = false;
        if (e < rows) {
          float c[12];
          fell = correction_row<kYs, kRows>(ys + lane, st_l1 + lane, st_om + lane, st_os + lane, cor.kappa, c);
          // h-mass of the correction: modes (a, b) = (0, 0) and (0, 1), i.e. 0 and 2
          m = st_mw[lane] * (double)c[2];
          float4 *cd = reinterpret_cast<float4 *>(cor.C + (size_t)e * 12);
#pragma unroll
          for (int k4 = 0; k4 < 3; ++k4) cd[k4] = make_float4(c[4 * k4], c[4 * k4 + 1], c[4 * k4 + 2], c[4 * k4 + 3]);
        }
        const unsigned long long fb = __ballot(fell);
        fell_count += (unsigned long long)__popcll(fb);
        any_fell = any_fell || fb != 0ull;
        // fixed-order (tree) wavefront sum of the tile's 64 masses, added in tile order
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m += __shfl_down(m, off, 64);
        mass += m;
      }
    }
  }
  if constexpr (FROM_Q) {
    if (wv == 0 && lane == 0) {
      cor.partial[blockIdx.x] = mass;
      if (cor.fallback && any_fell)
        atomicAdd(reinterpret_cast<unsigned long long *>(cor.fallback), fell_count);
    }
  }
}

int mlp_fused_blocks(int rows) {
  const int tiles = (rows + kRows - 1) / kRows;
  return tiles < kMlpGrid ? tiles : kMlpGrid;
}

hipError_t launch_mlp_fused(int dtype, const void *q, int n_lon, int n_lat, const float *fmean, const float *fistd,
                            const float *X, int rows, const __bf16 *W1f, const __bf16 *W2f, const __bf16 *W3t,
                            const float *b1, const float *b2, const float *b3p, float *Y, hipStream_t s,
                            const CorrectionArgs *ca) {
  static_assert(kInPad % 32 == 0 && kHidden == 32 * kWaves && kOutPad == 32 && kRows == 8 * kWaves,
                "fused network shape");
  if (rows <= 0) return hipSuccess;
  const dim3 grid(mlp_fused_blocks(rows)), block(64 * kWaves);
  if (!q) {
    hipLaunchKernelGGL((k_mlp_fused<float, false>), grid, block, 0, s, nullptr, 0, 0, nullptr, nullptr, X, rows, W1f,
                       W2f, W3t, b1, b2, b3p, Y, MlpCorrection<float>{});
    return hipGetLastError();
  }
  if (!ca) return hipErrorInvalidValue;
  if (dtype == 0) {
    MlpCorrection<double> c{static_cast<const double *>(ca->L1), ca->omean, ca->ostd, ca->mass_w, ca->kappa, ca->C,
                            ca->partial, ca->fallback};
    hipLaunchKernelGGL((k_mlp_fused<double, true>), grid, block, 0, s, static_cast<const double *>(q), n_lon, n_lat,
                       fmean, fistd, nullptr, rows, W1f, W2f, W3t, b1, b2, b3p, Y, c);
  } else {
    MlpCorrection<float> c{static_cast<const float *>(ca->L1), ca->omean, ca->ostd, ca->mass_w, ca->kappa, ca->C,
                           ca->partial, ca->fallback};
    hipLaunchKernelGGL((k_mlp_fused<float, true>), grid, block, 0, s, static_cast<const float *>(q), n_lon, n_lat,
                       fmean, fistd, nullptr, rows, W1f, W2f, W3t, b1, b2, b3p, Y, c);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ weights
// FP32 parameter vector -> BF16 operand copies, one launch for all of them
// (a launch costs more than any of the copies).  Fragment order of a matrix
// whose rows are MFMA A-operand rows and whose columns k are contracted: for
// rows [16 u, 16 u + 16) and columns [32 c, 32 c + 32) one 1 KB block,
// ((u K/32 + c) 64 + lane) 8 + j holding row 16 u + lane % 16 and column
// 32 c + 8 (lane / 16) + j, so that each load of a wavefront is one contiguous
// kilobyte.  Padded entries are zero.
__device__ __forceinline__ int frag_at(int row, int k, int K) {
  return ((row / 16) * (K / 32) + k / 32) * 512 + (row % 16 + 16 * ((k % 32) / 8)) * 8 + k % 8;
}

__global__ __launch_bounds__(256) void k_prep_weights(const float *__restrict__ P, PrepWeights w) {
  constexpr int n1 = kInPad * kHidden, n2 = kHidden * kHidden, n3 = kHidden * kOutPad;
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n1) {
    const int k = i / kHidden, n = i % kHidden;
    w.W1f[frag_at(n, k, kInPad)] = (__bf16)(k < kFeatures ? P[oW1 + (size_t)k * kHidden + n] : 0.0f);
    return;
  }
  i -= n1;
  if (i < n2) {
    const int k = i / kHidden, n = i % kHidden;
    const __bf16 v = (__bf16)P[oW2 + i];
    w.W2f[frag_at(n, k, kHidden)] = v;
    if (w.W2rf) w.W2rf[frag_at(k, n, kHidden)] = v;
    return;
  }
  i -= n2;
  if (i < n3) {
    const int k = i / kOutPad, n = i % kOutPad;
    const __bf16 v = (__bf16)(n < kOut ? P[oW3 + (size_t)k * kOut + n] : 0.0f);
    if (w.W3t) w.W3t[(size_t)n * kHidden + k] = v;
    if (w.W3f) w.W3f[frag_at(n, k, kHidden)] = v;
    if (w.W3rf) w.W3rf[frag_at(k, n, kOutPad)] = v;
    return;
  }
  i -= n3;
  if (i < kOutPad) w.b3p[i] = i < kOut ? P[ob3 + i] : 0.0f;
}

hipError_t launch_prep_weights(const float *P, const PrepWeights &w, hipStream_t s) {
  constexpr int total = kInPad * kHidden + kHidden * kHidden + kHidden * kOutPad + kOutPad;
  hipLaunchKernelGGL(k_prep_weights, dim3((total + 255) / 256), dim3(256), 0, s, P, w);
  return hipGetLastError();
}

// ------------------------------------------------------------------ training step
// One training step is three kernels after the weights' preparation:
//   k_train_rows    everything that is local to a row: both passes through the
//                   network for 32 rows per workgroup, activations in LDS,
//                   pre-activations in registers (the backward pass needs each
//                   in the lane that formed it); leaves the factors of the
//                   weight gradients in fragment order and the workgroup's
//                   sums of the bias gradients and of the squared error;
//   k_train_dw      the weight gradients, sums over the rows of activation x
//                   gradient, split over ranges of rows;
//   k_train_update  the ranges' sums in order, and Adam.
// The 29 launches this replaces (one GEMM, conversion, column sum or copy
// each) took 156 us at 8192 rows, launches and memory round trips almost all of
// it; these take 33.7.  Under the tracer, which lengthens every launch: rows 18.4
// (one tile per CU: a serial chain of five products and their barriers; the vector
// unit busy 0.23 of the time, waiting 0.49), gradients 9.2, update 5.3, weights 3.4.
// Rounding points as before: BF16 factors of every product, FP32
// accumulation, bias, GELU, loss and gradients in FP32.
constexpr int kTrRows = 32;               // rows of a tile: one K block of the weight gradients
constexpr int kLdX = kInPad + 8, kLdY = kOutPad + 8;   // LDS row strides in BF16

// acc[nt][mt] of this wavefront's units [32 wv, +32) = W in^T over K inputs, A
// fragments w, rows of `in` (stride ld) as B.
template <int K>
__device__ __forceinline__ void train_product(const bf16x8 (&w)[K / 32][2], const __bf16 *in, int ld, int lane,
                                              f32x4 (&acc)[2][2]) {
  const int r = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < K / 32; ++ks) {
    bf16x8 b[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) b[mt] = *reinterpret_cast<const bf16x8 *>(in + (16 * mt + r) * ld + 32 * ks + kq);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt], b[mt], acc[nt][mt], 0, 0, 0);
  }
}

template <int K>
__device__ __forceinline__ void train_weights(const __bf16 *__restrict__ Wf, int wv, int lane, bf16x8 (&w)[K / 32][2]) {
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks)
      w[ks][nt] = *reinterpret_cast<const bf16x8 *>(Wf + ((size_t)(2 * wv + nt) * (K / 32) + ks) * 512 + lane * 8);
}

// out = BF16(gelu(z + bias)) into LDS rows of stride kLd; z becomes gelu'.
__device__ __forceinline__ void train_gelu(f32x4 (&z)[2][2], const float *__restrict__ bias, __bf16 *out, int wv,
                                           int lane) {
  const int r = lane & 15;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int n0 = 32 * wv + 16 * nt + (lane >> 4) * 4;
    const float b[4] = {bias[n0], bias[n0 + 1], bias[n0 + 2], bias[n0 + 3]};
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float zi = z[nt][mt][i] + b[i];
        h[i] = (__bf16)gelu_and_grad(zi);
        z[nt][mt][i] = zi;
      }
      *reinterpret_cast<bf16x4 *>(out + (16 * mt + r) * kLd + n0) = h;
    }
  }
}

// Sum over the 16 lanes of a row group, in every lane of it, by rotations within
// the group (the vector unit's own lane moves: the LDS permutes of __shfl_xor
// are a round trip each; the pairs added are the same).
template <int ROT>
__device__ __forceinline__ float add_rotated(float t) {
  return t + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x120 + ROT, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum16(float t) {
  return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(t))));
}

// d = acc gelu' as BF16 into LDS; its sum over the tile's rows added to db
// (lanes of one 16-lane group hold the rows of a unit; lane % 16 == 0 the sum).
__device__ __forceinline__ void train_gelu_grad(const f32x4 (&acc)[2][2], const f32x4 (&gp)[2][2], __bf16 *out, int wv,
                                                int lane, float (&db)[2][4]) {
  const int r = lane & 15;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int n0 = 32 * wv + 16 * nt + (lane >> 4) * 4;
    float d[2][4];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d[mt][i] = acc[nt][mt][i] * gp[nt][mt][i];
        h[i] = (__bf16)d[mt][i];
      }
      *reinterpret_cast<bf16x4 *>(out + (16 * mt + r) * kLd + n0) = h;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      db[nt][i] += sum16(d[0][i] + d[1][i]);
    }
  }
}

// A tile's factor in[32 rows][units] to fragment order (the rows contracted):
// block u of the tile, 16 units, is one contiguous kilobyte.
__device__ __forceinline__ void train_fragments(const __bf16 *in, int ld, int units, __bf16 *__restrict__ out, int wv,
                                                int lane) {
  const int r = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll 2
  for (int u = wv; u < units / 16; u += kWaves) {
    bf16x8 f;
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = in[(kq + j) * ld + 16 * u + r];
    *reinterpret_cast<bf16x8 *>(out + (size_t)u * 512 + lane * 8) = f;
  }
}

__global__ __attribute__((amdgpu_waves_per_eu(2))) __launch_bounds__(64 * kWaves) void k_train_rows(TrainRows a) {
  __shared__ __attribute__((aligned(16))) __bf16 sx[kTrRows * kLdX];
  __shared__ __attribute__((aligned(16))) __bf16 sh1[kTrRows * kLd], sh2[kTrRows * kLd];
  __shared__ __attribute__((aligned(16))) __bf16 sd1[kTrRows * kLd], sd2[kTrRows * kLd];
  __shared__ __attribute__((aligned(16))) __bf16 sdy[kTrRows * kLdY];
  __shared__ float sse[kWaves];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float db1[2][4], db2[2][4], db3[4], se = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    db1[0][i] = db1[1][i] = db2[0][i] = db2[1][i] = 0.f;
    db3[i] = 0.f;
  }
  const int tiles = a.rows / kTrRows;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    // unknown to the compiler in every round, or it computes all of a round's
    // addresses before the loop and spills them
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, r = lane & 15;
    const size_t row0 = (size_t)tile * kTrRows;
    bf16x8 w1[kInPad / 32][2], w2[kHidden / 32][2];
    // inputs (any alignment of X), then the first layer's weights: loads complete
    // in order, and more of them in front of the LDS stores would hold those back
    float xv[(kTrRows * kFeatures + 64 * kWaves - 1) / (64 * kWaves)];
#pragma unroll
    for (int n = 0; n < (int)(sizeof(xv) / sizeof(float)); ++n) {
      const int idx = tid + 64 * kWaves * n;
      xv[n] = idx < kTrRows * kFeatures ? a.X[row0 * kFeatures + idx] : 0.f;
    }
    train_weights<kInPad>(a.w.W1f, wv, lane, w1);
#pragma unroll
    for (int n = 0; n < (int)(sizeof(xv) / sizeof(float)); ++n) {
      const int idx = tid + 64 * kWaves * n;
      if (idx < kTrRows * kFeatures) sx[(idx / kFeatures) * kLdX + idx % kFeatures] = (__bf16)xv[n];
    }
    for (int idx = tid; idx < kTrRows * (kInPad - kFeatures); idx += 64 * kWaves)
      sx[(idx / (kInPad - kFeatures)) * kLdX + kFeatures + idx % (kInPad - kFeatures)] = (__bf16)0.f;
    __syncthreads();
    f32x4 z1[2][2], z2[2][2], acc[2][2];
    train_product<kInPad>(w1, sx, kLdX, lane, z1);
    train_weights<kHidden>(a.w.W2f, wv, lane, w2);
    train_gelu(z1, a.P + ob1, sh1, wv, lane);
    __syncthreads();
    train_product<kHidden>(w2, sh1, kLd, lane, z2);
    // output layer, loss and its gradient: wavefront 2 mt + nt < 4 takes 16
    // rows x 16 outputs; the weights it and the way back need are requested
    // ahead of their barriers
    const int mt = (wv >> 1) & 1, nt = wv & 1, kq = (lane >> 4) * 8, n0 = 16 * nt + (lane >> 4) * 4;
    bf16x8 w3r[1][2], w3[kHidden / 32];
    float tv[4], b3[4];
#pragma unroll
    for (int ks = 0; ks < kHidden / 32; ++ks)
      w3[ks] = *reinterpret_cast<const bf16x8 *>(a.w.W3f + ((size_t)nt * (kHidden / 32) + ks) * 512 + lane * 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      tv[i] = n0 + i < kOut ? a.T[(row0 + 16 * mt + r) * kOut + n0 + i] : 0.f;
      b3[i] = a.w.b3p[n0 + i];
    }
    train_weights<kOutPad>(a.w.W3rf, wv, lane, w3r);
    train_gelu(z2, a.P + ob2, sh2, wv, lane);
    __syncthreads();
    if (wv < 4) {
      f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < kHidden / 32; ++ks) {
        const bf16x8 b = *reinterpret_cast<const bf16x8 *>(sh2 + (16 * mt + r) * kLd + 32 * ks + kq);
        y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3[ks], b, y, 0, 0, 0);
      }
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float g = 0.f;
        if (n0 + i < kOut && ((a.mask_bits >> (n0 + i)) & 1u)) {
          const float d = (y[i] + b3[i]) - tv[i];
          se += d * d;
          g = 2.f * d * a.scale;
        }
        h[i] = (__bf16)g;
        db3[i] += sum16(g);
      }
      *reinterpret_cast<bf16x4 *>(sdy + (16 * mt + r) * kLdY + n0) = h;
    }
    train_weights<kHidden>(a.w.W2rf, wv, lane, w2);
    __syncthreads();
    train_product<kOutPad>(w3r, sdy, kLdY, lane, acc);
    train_gelu_grad(acc, z2, sd2, wv, lane, db2);
    __syncthreads();
    train_product<kHidden>(w2, sd2, kLd, lane, acc);
    train_gelu_grad(acc, z1, sd1, wv, lane, db1);
    train_fragments(sx, kLdX, kInPad, a.Xf + row0 * kInPad, wv, lane);
    train_fragments(sh1, kLd, kHidden, a.H1f + row0 * kHidden, wv, lane);
    train_fragments(sh2, kLd, kHidden, a.H2f + row0 * kHidden, wv, lane);
    train_fragments(sd2, kLd, kHidden, a.D2f + row0 * kHidden, wv, lane);
    train_fragments(sdy, kLdY, kOutPad, a.DYf + row0 * kOutPad, wv, lane);
    __syncthreads();
    train_fragments(sd1, kLd, kHidden, a.D1f + row0 * kHidden, wv, lane);
    __syncthreads();          // the next tile overwrites the LDS arrays
  }
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15;
  // this workgroup's sums: [b1 | b2 | b3 of rows 0..15 | .. of rows 16..31], squared error
  float *bp = a.bias_part + (size_t)blockIdx.x * kBiasPart;
  if (r == 0) {
    const int n0 = 32 * wv + (lane >> 4) * 4;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bp[n0 + 16 * nt + i] = db1[nt][i];
        bp[kHidden + n0 + 16 * nt + i] = db2[nt][i];
      }
    if (wv < 4)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        bp[2 * kHidden + kOutPad * (wv >> 1) + 16 * (wv & 1) + (lane >> 4) * 4 + i] = db3[i];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off, 64);
  if (lane == 0) sse[wv] = se;
  __syncthreads();
  if (tid == 0) a.se_part[blockIdx.x] = (sse[0] + sse[1]) + (sse[2] + sse[3]);
}

int train_row_blocks(int rows) {
  const int t = rows / kTrRows;
  return t < kMaxTrainBlocks ? t : kMaxTrainBlocks;
}

// Weight gradients: a wavefront takes 32 x 64 outputs (32 x 32 of the output
// layer's) of one matrix over one range of rows, block of 32 rows by block (six
// fragments of a kilobyte, eight MFMAs each).  The four wavefronts of a
// workgroup share the activations (of the output layer's: the gradients); 14
// workgroups a range: 8 of W2, 4 of W1, 2 of W3.  The fragments come from other
// XCDs' caches, so latency bounds it: four blocks' loads are in flight at once,
// and a range belongs to one XCD.  Ranges of 256 rows, each summed in order and
// then the ranges in order, fix the bits of the gradients.  8192 rows: 8.9 us
// (10.2 with 64 x 64 outputs a wavefront; with ranges of 512 rows split over the
// wavefronts of a workgroup 8.7).
constexpr int kDwWaves = 4, kDwJobs = 14;

template <int NT>
__device__ __forceinline__ void train_dw(const __bf16 *__restrict__ A, int ua, const __bf16 *__restrict__ B, int ub,
                                         int c0, int c1, int lane, float *__restrict__ C, int ldc) {
  constexpr int MT = 2;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int c = c0; c < c1; ++c) {
    bf16x8 a[MT], b[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const bf16x8 *>(A + ((size_t)c * ua + i) * 512 + lane * 8);
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = *reinterpret_cast<const bf16x8 *>(B + ((size_t)c * ub + j) * 512 + lane * 8);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) C[(size_t)(16 * i + (lane >> 4) * 4 + e) * ldc + 16 * j + (lane & 15)] = acc[i][j][e];
}

__global__ __launch_bounds__(64 * kDwWaves) void k_train_dw(TrainDw a) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroups are dispatched round-robin over the 8 XCDs: each takes a
  // contiguous run of (range, job), so a range's rows are read by one XCD
  const int nb = gridDim.x, x = blockIdx.x & 7, nx = nb >> 3, rem = nb & 7;
  const int id = x * nx + (x < rem ? x : rem) + (blockIdx.x >> 3);
  const int range = id / kDwJobs, job = id - range * kDwJobs;
  const int c0 = range * a.per, c1 = c0 + a.per < a.chunks ? c0 + a.per : a.chunks;
  float *G = a.part + (size_t)range * kGradPart;
  constexpr int UH = kHidden / 16, UX = kInPad / 16, UY = kOutPad / 16;
  static_assert(kHidden == 64 * kDwWaves && kHidden == 8 * 32 && kInPad == 4 * 32 && kOutPad == 32, "jobs");
  if (job < 8) {
    train_dw<4>(a.H1f + job * 2 * 512, UH, a.D2f + wv * 4 * 512, UH, c0, c1, lane,
                G + oG2 + (size_t)job * 32 * kHidden + wv * 64, kHidden);
  } else if (job < 12) {
    const int m = job - 8;
    train_dw<4>(a.Xf + m * 2 * 512, UX, a.D1f + wv * 4 * 512, UH, c0, c1, lane,
                G + oG1 + (size_t)m * 32 * kHidden + wv * 64, kHidden);
  } else {
    const int m = (job - 12) * kDwWaves + wv;
    train_dw<2>(a.H2f + m * 2 * 512, UH, a.DYf, UY, c0, c1, lane, G + oG3 + (size_t)m * 32 * kOutPad, kOutPad);
  }
}

int train_splits(int rows) {
  const int s = (rows + 255) / 256;
  return s < 1 ? 1 : (s > kMaxSplits ? kMaxSplits : s);
}

// Gradients and Adam, a thread per weight (the ranges' sums added in order);
// the biases by 32 threads each over the workgroups' sums, in blocks of their
// own; the last block the loss.
__device__ __forceinline__ void train_param(const TrainUpdate &a, int i, float g) {
  if (a.grads) a.grads[i] = g;
  if (a.lr > 0.f) {
    const float mi = a.b1 * a.m[i] + (1.f - a.b1) * g;
    const float vi = a.b2 * a.v[i] + (1.f - a.b2) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    a.p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  }
}

constexpr int kUpW1 = kFeatures * kHidden / 256, kUpW2 = kHidden * kHidden / 256, kUpW3 = kHidden * kOut / 256;
constexpr int kUpB = (2 * kHidden + kOutPad) / 8;       // 8 biases per block, 32 threads each

__global__ __launch_bounds__(256) void k_train_update(TrainUpdate a) {
  __shared__ float sh[256];
  const int t = threadIdx.x;
  int b = blockIdx.x;
  if (b < kUpW1 + kUpW2 + kUpW3) {
    int i, o;                                           // parameter, place in a range's sums
    if (b < kUpW1) {
      const int n = b * 256 + t;
      i = (int)oW1 + n;
      o = oG1 + n;
    } else if (b < kUpW1 + kUpW2) {
      const int n = (b - kUpW1) * 256 + t;
      i = (int)oW2 + n;
      o = oG2 + n;
    } else {
      const int n = (b - kUpW1 - kUpW2) * 256 + t;
      i = (int)oW3 + n;
      o = oG3 + n / kOut * kOutPad + n % kOut;
    }
    const float *p = a.part + o;
    float g = 0.f;
#pragma unroll 16
    for (int z = 0; z < a.splits; ++z) g += p[(size_t)z * kGradPart];
    train_param(a, i, g);
    return;
  }
  b -= kUpW1 + kUpW2 + kUpW3;
  if (b < kUpB) {
    const int j = b * 8 + (t & 7);                      // of b1, b2, b3 (padded)
    float g = 0.f;
#pragma unroll 8
    for (int k = t >> 3; k < a.blocks; k += 32) {
      const float *p = a.bias_part + (size_t)k * kBiasPart + j;
      g += j < 2 * kHidden ? p[0] : p[0] + p[kOutPad];
    }
    sh[t] = g;
    __syncthreads();
    for (int off = 128; off >= 8; off >>= 1) {
      if (t < off) sh[t] += sh[t + off];
      __syncthreads();
    }
    if (t >= 8) return;
    if (j < kHidden) train_param(a, (int)ob1 + j, sh[t]);
    else if (j < 2 * kHidden) train_param(a, (int)ob2 + j - kHidden, sh[t]);
    else if (j < 2 * kHidden + kOut) train_param(a, (int)ob3 + j - 2 * kHidden, sh[t]);
    return;
  }
  float se = 0.f;
  for (int k = t; k < a.blocks; k += 256) se += a.se_part[k];
  sh[t] = se;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (t < off) sh[t] += sh[t + off];
    __syncthreads();
  }
  if (t == 0) *a.loss = a.scale * sh[0];
}

hipError_t launch_train(const TrainRows &r, const TrainDw &d, const TrainUpdate &u, hipStream_t s) {
  static_assert(kUpW1 * 256 == kFeatures * kHidden && kUpW2 * 256 == kHidden * kHidden && kUpW3 * 256 == kHidden * kOut &&
                    kUpB * 8 == 2 * kHidden + kOutPad,
                "update blocks");
  hipLaunchKernelGGL(k_train_rows, dim3(u.blocks), dim3(64 * kWaves), 0, s, r);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_train_dw, dim3(kDwJobs * u.splits), dim3(64 * kDwWaves), 0, s, d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_train_update, dim3(kUpW1 + kUpW2 + kUpW3 + kUpB + (u.loss ? 1 : 0)), dim3(256), 0, s, u);
  return hipGetLastError();
}

// The real columns of a padded matrix G[k_in][np_] into out[k_in][n_out].
__global__ void k_unpad(const float *__restrict__ G, int k_in, int n_out, int np_, float *__restrict__ out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= k_in * n_out) return;
  const int k = idx / n_out, n = idx - k * n_out;
  out[idx] = G[(size_t)k * np_ + n];
}

hipError_t launch_unpad(const float *G, int k_in, int n_out, int np_, float *out, hipStream_t s) {
  const int total = k_in * n_out;
  hipLaunchKernelGGL(k_unpad, dim3((total + 255) / 256), dim3(256), 0, s, G, k_in, n_out, np_, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ features
// X[e][k] = (q1[nb(e, k)][v][m] - mean[k]) * istd[k] for the 3 x 3 stencil of
// an r = 1 state (periodic in longitude, pole row repeated across a pole),
// k = ((dj+1)*3 + (di+1))*12 + v*4 + m, FP32, not standardised without
// mean/istd.  Bound by its 432 bytes of output per element: a thread makes four
// consecutive values (they share a stencil neighbour, so the index arithmetic
// and its division are paid once for four) and stores them at once.  64 800
// elements, 28 MB: 18.8 us with one value per thread, now 9.4 us.
struct __attribute__((aligned(4))) Float4u { float x[4]; };
template <typename T>
__global__ __launch_bounds__(256) void k_features_f32(const T *__restrict__ q, int n_lon, int n_lat,
                                                      const float *__restrict__ mean,
                                                      const float *__restrict__ istd, float *__restrict__ X) {
  constexpr int kQuads = kFeatures / 4;
  static_assert(kFeatures % 4 == 0 && 12 % 4 == 0, "four values of one neighbour");
  const size_t first = (size_t)blockIdx.x * 256;
  const size_t eb = first / kQuads;
  const int local = (int)(first - eb * kQuads) + (int)threadIdx.x;
  const int de = local / kQuads, c = local - de * kQuads;
  if (eb + de >= (size_t)n_lon * n_lat) return;
  const int e = (int)eb + de;
  const int s = c / 3, vm = 4 * (c - s * 3);
  const int dj = s / 3 - 1, di = s % 3 - 1;
  const int j = e / n_lon, i = e - j * n_lon;
  int jj = j + dj;
  jj = jj < 0 ? 0 : (jj >= n_lat ? n_lat - 1 : jj);
  int ii = i + di;
  ii = ii < 0 ? ii + n_lon : (ii >= n_lon ? ii - n_lon : ii);
  const T *src = q + ((size_t)jj * n_lon + ii) * 12 + vm;
  Float4u o;
#pragma unroll
  for (int k = 0; k < 4; ++k) o.x[k] = (float)src[k];
  if (mean) {
#pragma unroll
    for (int k = 0; k < 4; ++k) o.x[k] = (o.x[k] - mean[4 * c + k]) * istd[4 * c + k];
  }
  *reinterpret_cast<Float4u *>(X + (size_t)e * kFeatures + 4 * c) = o;
}

hipError_t launch_features_f32(int dtype, const void *q, int n_lon, int n_lat, const float *mean, const float *istd,
                               float *X, hipStream_t s) {
  const size_t total = (size_t)n_lon * n_lat * (kFeatures / 4);
  const dim3 grid((unsigned)((total + 255) / 256));
  if (dtype == 0)
    hipLaunchKernelGGL(k_features_f32<double>, grid, dim3(256), 0, s, static_cast<const double *>(q), n_lon, n_lat,
                       mean, istd, X);
  else
    hipLaunchKernelGGL(k_features_f32<float>, grid, dim3(256), 0, s, static_cast<const float *>(q), n_lon, n_lat,
                       mean, istd, X);
  return hipGetLastError();
}

// ------------------------------------------------------------------ learned stage
// delta = -(sum of partials) / (sum over elements of mass_w[j][0]): the mode-00
// h-correction that makes the total h-mass change of the correction zero.
// Every block of the output kernel forms it itself, in the same fixed order.
__device__ __forceinline__ double block_mass_delta(const double *__restrict__ partial, int nparts, double area,
                                                  double *sh) {
  double acc = 0.0;
  for (int k = threadIdx.x; k < nparts; k += 256) acc += partial[k];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  return -sh[0] / area;
}

// out = combine ? c0 q0 + c1 (q + dt (L1 + c)) : L1 + c, with c_(h,00) = delta;
// the combination is evaluated as y + c0 (q0 - y) + ce y, y = q + dt (L1 + c),
// ce = c0 + c1 - 1 formed in FP64, so the weights sum to one exactly.
template <typename T>
__global__ __launch_bounds__(256) void k_learned_out(const T *__restrict__ q, const T *q0, const T *__restrict__ L1,
                                                     const float *__restrict__ C, const double *__restrict__ partial,
                                                     int nparts, double area, int E, int combine, T c0, T ce, T dt,
                                                     T *out) {
  __shared__ double sh[256];
  // the element's operands first, so that their loads are in flight while
  // the block sums the mass partials (the same arithmetic either way)
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const bool live = idx < E * 12;
  const int k = idx % 12;
  T l1v = T(0), qv = T(0), qn = T(0);
  float cv = 0.f;
  if (live) {
    l1v = L1[idx];
    if (k != 0) cv = C[idx];
    if (combine) {
      qv = q[idx];
      if (c0 != T(0)) qn = q0[idx];
    }
  }
  const double delta = block_mass_delta(partial, nparts, area, sh);
  if (!live) return;
  const T corr = k == 0 ? (T)delta : (T)cv;
  const T l = l1v + corr;
  if (combine) {
    const T y = qv + dt * l;
    out[idx] = y + c0 * (qn - y) + ce * y;
  } else {
    out[idx] = l;
  }
}

hipError_t launch_learned_out(int dtype, const LearnedOut &a, hipStream_t s) {
  const int ob = (a.E * 12 + 255) / 256;
  if (dtype == 0)
    hipLaunchKernelGGL(k_learned_out<double>, dim3(ob), dim3(256), 0, s, static_cast<const double *>(a.q),
                       static_cast<const double *>(a.q0), static_cast<const double *>(a.L1), a.C, a.partial, a.nparts,
                       a.area, a.E, a.combine, a.c0, a.c0 + a.c1 - 1.0, a.dt, static_cast<double *>(a.out));
  else
    hipLaunchKernelGGL(k_learned_out<float>, dim3(ob), dim3(256), 0, s, static_cast<const float *>(a.q),
                       static_cast<const float *>(a.q0), static_cast<const float *>(a.L1), a.C, a.partial, a.nparts,
                       a.area, a.E, a.combine, (float)a.c0, (float)(a.c0 + a.c1 - 1.0), (float)a.dt,
                       static_cast<float *>(a.out));
  return hipGetLastError();
}

// ------------------------------------------------------------------ projection
// Cos-weighted L2 projection of an order-r state onto order k on the same
// mesh: the longitude degrees a <= min(k, r) are kept (orthonormal, the mass
// matrix is diagonal in a), the latitude degrees mix through the per-row
// (k+1) x (r+1) matrix Pj[b'][b].  Bound by the source state.  A thread makes
// the k+1 outputs of one (element, variable, a), its source values read once
// and all at the start, and a workgroup's elements share a latitude, so that
// the matrix comes through the scalar cache.  64 800 FP64 elements, r = 4 to 1,
// 45 MB: 10.3 us with one output per thread, now 8.3 us (with a
// loop of runtime length, one load in flight per thread, 11.5 us).
// STAGED: the values that are used come through LDS, read in memory order.  A
// thread's own reads, nk values of every row, go over each cache line several
// times, which costs most where rows are short and little of them is used: up
// to half of it in FP32 and a fifth in FP64 (us for 720x360 elements, direct /
// staged / one output per thread: FP32 r = 7 to 1 73.7 / 32.3 / 36.4, 7 to 3 50.6 /
// 43.4 / 79.7, 4 to 1 22.7 / 17.1 / 19.6, FP64 6 to 0 61.4 / 51.7 / 68.9); otherwise
// direct is as fast or faster (FP32 2 to 1 9.2 / 12.9, FP64 7 to 1 75.7 / 82.4).
template <typename T, int NP, bool STAGED>
__global__ __launch_bounds__(256) void k_project(const T *__restrict__ q, int n_lon, int nk, int bpr,
                                                 const double *__restrict__ P, T *__restrict__ out) {
  const int j = blockIdx.x / bpr;
  const int t0 = (blockIdx.x - j * bpr) * 256, t = t0 + threadIdx.x, all = n_lon * 3 * nk;
  const size_t row = (size_t)j * n_lon * 3;
  const int ev0 = t0 / nk;                                 // the block's first (element of the row, variable)
  // 256 threads cover at most 256 / nk + 2 of them, nk NP values each
  __shared__ T sx[STAGED ? (256 + 2 * NP) * NP : 1];
  if constexpr (STAGED) {
    const int ev1 = (t0 + 255 < all ? t0 + 255 : all - 1) / nk, used = nk * NP, count = (ev1 - ev0 + 1) * used;
    const T *src = q + (row + ev0) * (NP * NP);
    for (int k = threadIdx.x; k < count; k += 256) {
      const int ev = k / used, r = k - ev * used, b = r / nk;
      sx[k] = src[ev * (NP * NP) + b * NP + (r - b * nk)];
    }
    __syncthreads();
  }
  if (t >= all) return;
  const int ev = t / nk, a = t - ev * nk;                  // (element of the row, variable), a
  T x[NP];
  if constexpr (STAGED) {
#pragma unroll
    for (int b = 0; b < NP; ++b) x[b] = sx[((ev - ev0) * NP + b) * nk + a];
  } else {
    const T *qe = q + (row + ev) * (NP * NP) + a;
#pragma unroll
    for (int b = 0; b < NP; ++b) x[b] = a < NP ? qe[b * NP] : (T)0;
  }
  const double *Pj = P + (size_t)j * nk * NP;
  T *o = out + (row + ev) * nk * nk + a;
  for (int bp = 0; bp < nk; ++bp) {
    double acc = 0.0;
#pragma unroll
    for (int b = 0; b < NP; ++b) acc += Pj[bp * NP + b] * (double)x[b];
    o[bp * nk] = (T)acc;
  }
}

template <typename T>
static hipError_t launch_project_t(const T *q, int n_lon, int n_lat, int np, int nk, const double *P, T *out,
                                   hipStream_t s) {
  const int bpr = (int)(((long long)n_lon * 3 * nk + 255) / 256);
  const dim3 grid((unsigned)((long long)bpr * n_lat)), block(256);
  constexpr int kPart = sizeof(T) == 4 ? 2 : 5;
  const bool staged = nk * kPart <= np;
  switch (np) {
#define DGSW_PROJECT(NP)                                                                               \
  case NP:                                                                                             \
    if constexpr (NP >= kPart)                                                                         \
      if (staged) {                                                                                    \
        hipLaunchKernelGGL((k_project<T, NP, true>), grid, block, 0, s, q, n_lon, nk, bpr, P, out);    \
        break;                                                                                         \
      }                                                                                                \
    hipLaunchKernelGGL((k_project<T, NP, false>), grid, block, 0, s, q, n_lon, nk, bpr, P, out);       \
    break
    DGSW_PROJECT(1); DGSW_PROJECT(2); DGSW_PROJECT(3); DGSW_PROJECT(4);
    DGSW_PROJECT(5); DGSW_PROJECT(6); DGSW_PROJECT(7); DGSW_PROJECT(8);
#undef DGSW_PROJECT
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_project(int dtype, const void *q, int n_lon, int E, int np, int nk, const double *P,
                          void *out, hipStream_t s) {
  const int n_lat = E / n_lon;
  return dtype == 0 ? launch_project_t(static_cast<const double *>(q), n_lon, n_lat, np, nk, P,
                                       static_cast<double *>(out), s)
                    : launch_project_t(static_cast<const float *>(q), n_lon, n_lat, np, nk, P,
                                       static_cast<float *>(out), s);
}

}  // namespace dgsw
