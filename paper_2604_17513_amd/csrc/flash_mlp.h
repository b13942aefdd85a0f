// Learned warm start network: shapes, parameter layout and launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "flash_device.h"

namespace flash {

constexpr int kFeat = 16;      // per-contact input features
constexpr int kHidden = 128;   // width of the three hidden layers
constexpr int kOut = 3;        // (n, t1, t2) multiplier prediction
constexpr int kNorm = 2 * kFeat + kOut;   // feature means, feature inverse scales, label scales

// Parameters packed as W1, b1, W2, b2, W3, b3, W4, b4; W row-major (out x in).
struct MlpLayout {
  static constexpr long w1 = 0;
  static constexpr long b1 = w1 + (long)kHidden * kFeat;
  static constexpr long w2 = b1 + kHidden;
  static constexpr long b2 = w2 + (long)kHidden * kHidden;
  static constexpr long w3 = b2 + kHidden;
  static constexpr long b3 = w3 + (long)kHidden * kHidden;
  static constexpr long w4 = b3 + kHidden;
  static constexpr long b4 = w4 + (long)kOut * kHidden;
  static constexpr long total = b4 + kOut;
};
static_assert(MlpLayout::total == 35587, "parameter count");

// Gradient slabs: a workgroup of the gradient kernel takes grad_span(rows) rows at a time and sums into a slab of
// its own.  At most one workgroup per CU (its LDS), so at most kMaxSlabs slabs; up to 256 rows go into one sum,
// and more are split evenly.
constexpr long kGradRows = 128;
constexpr long kMaxSlabs = 256;
constexpr long kSlab = (MlpLayout::total + 3) / 4 * 4;
inline int grad_span(long rows) {
  const long b = (rows + kGradRows - 1) / kGradRows;
  if (b <= 2 || b > kMaxSlabs) return (int)kGradRows;
  return (int)(((rows + b - 1) / b + 7) / 8 * 8);
}
inline long grad_slabs(long rows) {
  if (rows <= 2 * kGradRows) return 1;
  const long span = grad_span(rows), b = (rows + span - 1) / span;
  return b < kMaxSlabs ? b : kMaxSlabs;
}
// Scratch of one gradient of up to `rows` rows: grad_slabs slabs and doubles, and dz of three layers and of the
// output per row.
struct GradScratch {
  float* slab;
  double* partial;
  float* dz;        // [3][kHidden / 4][rows][4], 16-byte aligned
  float* dy;        // [rows][kOut]
};

// Device buffers of an inference pass over the contact slots of a batch.
struct MlpBuffers {
  const float* W;      // FP32 copy of the bf16 weights (exactly representable)
  const float* norm;   // [kNorm]
  float* feat;         // [rows * kFeat] raw features
  int* need;           // [rows] 1: active contact without a previous-step multiplier
  float* Y;            // [rows * kOut]
  double* lam_ml;      // [rows * 3] cone-projected candidate multipliers
};

// Raises the dynamic LDS limits of the network kernels (call once before their first launch).
void prepare_mlp();
// Fused forward pass on the matrix cores: Y = network(X).  norm != nullptr: X holds raw
// features; need != nullptr: 32-row tiles without a flagged row are skipped.
void launch_mlp_fused(const float* W, const float* norm, const float* X, long rows, const int* need, float* Y,
                      hipStream_t s);
// Mean squared loss of rows (X, Lab) and its gradient.
void launch_mlp_grad(const float* W, const float* X, const float* Lab, long rows, float* grad, float* loss,
                     const GradScratch& g, hipStream_t s);
// One minibatch of training: rows idx of the raw features and labels, normalised with norm; Adam step t on
// W, m, v; the loss before the step.
void launch_mlp_train(float* W, const float* norm, const float* feat, const float* lab, const int* idx, long rows,
                      float* m, float* v, float lr, int t, float* loss, const GradScratch& g, hipStream_t s);
void mlp_loss(const float* Y, const float* Lab, long n, double* partial, float* loss, hipStream_t s);
void launch_gather_batch(const float* feat, const float* lab, const int* idx, int B, const float* norm, float* X,
                         float* Y, hipStream_t s);
void launch_col_moments(const float* X, long rows, int cols, double* out, hipStream_t s);

template <class T> void launch_ws_features(const DevBatch<T>& B, const T* mu_env, float* feat, int* need,
                                          hipStream_t s);
// labels of the first contact solve of a step (launched right after it)
template <class T> void launch_ws_labels(const DevBatch<T>& B, const float* feat, float* lab, hipStream_t s);
template <class T> void launch_ws_infer(const DevBatch<T>& B, const T* mu_env, const MlpBuffers& M, hipStream_t s);
// Appends the active contact slots' rows (feature, label) in env order; base = rows already stored.
// coff: device scratch of n_envs + 1 ints; coff[n_envs] receives the number of rows appended.
template <class T> void launch_ws_compact(const DevBatch<T>& B, const float* feat, const float* lab, float* out_feat,
                                         float* out_lab, long base, int* coff, hipStream_t s);

}  // namespace flash
