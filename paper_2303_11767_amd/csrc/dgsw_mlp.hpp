// Launchers of the learned-correction kernels (dgsw_mlp.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dgsw {

constexpr int kFeatures = 108;   // 3 x 3 stencil x 3 variables x 4 modes
constexpr int kHidden = 256;
constexpr int kOut = 12;         // 3 variables x 4 modes of r = 1
constexpr int kInPad = 128;      // feature width padded for the K loop
constexpr int kOutPad = 32;      // output width padded for the N tiles

// offsets into the flat FP32 parameter vector
constexpr int64_t kParams = (int64_t)kFeatures * kHidden + kHidden + (int64_t)kHidden * kHidden + kHidden +
                            (int64_t)kHidden * kOut + kOut;
constexpr int64_t oW1 = 0, ob1 = oW1 + (int64_t)kFeatures * kHidden, oW2 = ob1 + kHidden,
                  ob2 = oW2 + (int64_t)kHidden * kHidden, oW3 = ob2 + kHidden,
                  ob3 = oW3 + (int64_t)kHidden * kOut;

// The learned stage's correction step, fused into the network kernel.
struct CorrectionArgs {
  const void *L1;                // plain r = 1 right-hand side [E][12] (state dtype)
  const float *omean, *ostd;     // [n_lat][12]
  const double *mass_w;          // [n_lat][2]
  float kappa;
  float *C;                      // corrections [E][12]
  double *partial;               // one h-mass per workgroup: mlp_fused_blocks(E)
  int64_t *fallback;             // optional device counter (64-bit: never wraps)
};
// workgroups of the persistent network kernel for `rows` rows (at most one
// per compute unit)
int mlp_fused_blocks(int rows);
// Whole-network inference, tiles of 64 rows, activations in LDS.  With q:
// rows = elements of the r = 1 state q (dtype 0/1), features computed from q,
// then the correction of each element (ca required; Y unused).  With q == NULL:
// rows of X[rows][108] (FP32) -> Y[rows][32] FP32 (the first 12 used).  W1f,
// W2f: the hidden layers' weights in fragment order (launch_prep_weights' Wf),
// W3t: the output layer's as Wt.
hipError_t launch_mlp_fused(int dtype, const void *q, int n_lon, int n_lat, const float *fmean, const float *fistd,
                            const float *X, int rows, const __bf16 *W1f, const __bf16 *W2f, const __bf16 *W3t,
                            const float *b1, const float *b2, const float *b3p, float *Y, hipStream_t s,
                            const CorrectionArgs *ca);
// BF16 copies of the weights (null: not made) and the padded output biases.
// *f: fragment order of the matrix whose rows are the layer's outputs, *rf:
// whose rows are its inputs (backward); W3t[output][input] row-major.
struct PrepWeights {
  __bf16 *W1f, *W2f, *W3t, *W3f, *W2rf, *W3rf;
  float *b3p;
};
hipError_t launch_prep_weights(const float *params, const PrepWeights &w, hipStream_t s);

// The training step (kernels in dgsw_mlp.hip).  Factors of the weight
// gradients, per 32 rows: blocks of 16 units in fragment order.
constexpr int kMaxTrainBlocks = 512;                       // workgroups of the row kernel
constexpr int kBiasPart = 2 * kHidden + 2 * kOutPad;       // a workgroup's bias-gradient sums
constexpr int kMaxSplits = 64;                             // ranges of rows of the weight gradients
constexpr int oG1 = 0, oG2 = kInPad * kHidden, oG3 = oG2 + kHidden * kHidden;
constexpr int kGradPart = oG3 + kHidden * kOutPad;         // a range's weight-gradient sums
int train_row_blocks(int rows);
int train_splits(int rows);
struct TrainRows {
  const float *P, *X, *T;
  int rows;
  unsigned mask_bits;       // bit n: output n counts
  float scale;              // 1 / (rows x outputs that count)
  PrepWeights w;
  __bf16 *Xf, *H1f, *H2f, *DYf, *D2f, *D1f;
  float *bias_part, *se_part;
};
struct TrainDw {
  const __bf16 *Xf, *H1f, *H2f, *DYf, *D2f, *D1f;
  int chunks, per;          // 32-row chunks, and how many a range takes
  float *part;              // [splits][kGradPart]
};
struct TrainUpdate {
  const float *part, *bias_part, *se_part;
  int splits, blocks;
  float scale;
  float *grads, *loss;      // optional
  float *p, *m, *v;         // updated when lr > 0
  float lr, b1, b2, eps, c1, c2;
};
hipError_t launch_train(const TrainRows &r, const TrainDw &d, const TrainUpdate &u, hipStream_t s);
hipError_t launch_unpad(const float *G, int k_in, int n_out, int np_, float *out, hipStream_t s);
hipError_t launch_features_f32(int dtype, const void *q, int n_lon, int n_lat, const float *mean, const float *istd,
                               float *X, hipStream_t s);
hipError_t launch_project(int dtype, const void *q, int n_lon, int E, int np, int nk, const double *P,
                          void *out, hipStream_t s);

// The learned stage's last step: out = L1 + C, the (h, 00) entry replaced by
// the global h-mass delta formed from the per-workgroup partials, or the
// Runge-Kutta combination with it.
struct LearnedOut {
  const void *L1;        // plain r = 1 right-hand side [E][12]
  const float *C;        // corrections [E][12]
  const double *partial; // nparts per-workgroup h-masses of the corrections
  int nparts, E;
  double area;           // sum over elements of mass_w[j][0]
  const void *q, *q0;
  void *out;
  int combine;
  double c0, c1, dt;
};
hipError_t launch_learned_out(int dtype, const LearnedOut &a, hipStream_t s);

}  // namespace dgsw
