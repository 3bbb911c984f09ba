// mlp_ops.h -- host launchers of the multiplier-surrogate kernels (mlp.hip).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>

namespace lbm {

constexpr int MLP_PARAMS = 9176;     // packed master parameters (floats)
constexpr int MLP_TRAINABLE = 9160;  // all but the output de-normalisation

void mlp_operands(const float *w, void *P, hipStream_t st);
// training set of n raw samples x [n][4] and labels lam [n][8] (device, mapped
// to the canonical octant in place): the labels' mean and deviation into
// stats [16] and the packed parameters w, the normalised inputs and targets
// into xh [n][4], th [n][8]; part: mlp_prepare_bytes(n) - 16 doubles
void mlp_prepare(double *x, double *lam, int64_t n, double *part, double *stats, float *w, float *xh, float *th,
                 hipStream_t st);
size_t mlp_prepare_bytes(int64_t n);
// gradient (written to grad[MLP_TRAINABLE]) and loss (added to *loss) of
// count samples (a multiple of 32); gpart: mlp_partials_bytes(count) of
// device scratch
void mlp_grad_batch(const void *P, const float *xh, const float *th, const int32_t *perm, int64_t count,
                    float *gpart, float *grad, float *loss, hipStream_t st);
// one Adam step t = 1, 2, ... on the gradient of the samples perm[off ..
// off + count)
void mlp_train_batch(void *P, const float *xh, const float *th, const int32_t *perm, int64_t off, int64_t count,
                     float *gpart, float *loss, float *w, float *m, float *v, float lr, int t, hipStream_t st);
size_t mlp_partials_bytes(int64_t count);
void mlp_predict(const void *P, const double *x, int64_t n, double *lam, hipStream_t st);
void mlp_label(const double *x, int64_t n, double tol, int max_it, double *lam, uint8_t *ok, int *iters,
               hipStream_t st);
size_t mlp_operands_bytes();

}  // namespace lbm
