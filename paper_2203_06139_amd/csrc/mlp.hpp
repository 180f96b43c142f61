// mlp.hpp -- kernels of the learned initialiser (mlp.hip, mlp_net.hip) and the
// network's parameter and workspace layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hf {

constexpr int kMlpIn = 256;
constexpr int kMlpHidden = 512;
constexpr int kMlpOut = 5;
constexpr int kMlpOutPad = 32;

hipError_t rebin_lognorm(int B, const void* counts, int dtype, const int64_t* offsets, float mean,
                         float std, float* out, hipStream_t s);
hipError_t default_starts(int B, const void* counts, int dtype, const int64_t* offsets,
                          const double* ranges, double t_shift, double t_scale, double* theta0,
                          hipStream_t s);
hipError_t theta_to_target(int B, const double* th, const float* mean, const float* std, float* t,
                           hipStream_t s);
hipError_t target_to_theta(int B, const float* y, const float* mean, const float* std, double* th,
                           hipStream_t s);
hipError_t column_stats(int64_t n, int cols, const float* x, float* mean, float* stdv,
                        hipStream_t s);

// Parameter layout (offsets in floats) and workspace carving.
struct MlpLayout {
  static constexpr int64_t kW[4] = {0, 131584, 394240, 656896};
  static constexpr int64_t kB[4] = {131072, 393728, 656384, 673280};
  static constexpr int kIn[4] = {kMlpIn, kMlpHidden, kMlpHidden, kMlpHidden};
  static constexpr int kOutDim[4] = {kMlpHidden, kMlpHidden, kMlpHidden, kMlpOutPad};
  static constexpr int64_t kTotal = 673312;
};

struct MlpWorkspace {
  uint16_t* a[4];   // a[0] = x, a[1..3] hidden activations, [B][in]
  uint16_t* at[4];  // the same in fragment order, K = rows (see mlp_net.hip)
  float* z[4];      // z[1..3] hidden pre-activations [B][512]
  float* y;         // [B][32]
  uint16_t* dz[5];  // dz[1..4] layer adjoints [B][out]
  uint16_t* dzt[5]; // the same in fragment order, K = rows
  uint16_t* wb[4];  // layer weights bf16 in fragment order, K = inputs
  uint16_t* wt[4];  // in fragment order, K = outputs (wt[0] unused)
  double* loss_part;  // one partial sum of the loss per block of rows
};

int64_t mlp_workspace_bytes(int B);
MlpWorkspace mlp_carve(void* base, int B);
hipError_t mlp_forward(int B, const float* params, const float* x, float* y, void* ws, hipStream_t s);
hipError_t mlp_train_step(int B, float* params, float* m, float* v, int step, float lr, float wd,
                          const float* x, const float* t, float* grads, float* loss, void* ws,
                          hipStream_t s);

}  // namespace hf
