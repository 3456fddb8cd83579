// Launchers of the layer kernels in conv.hip and wgrad.hip, used by the layer entry points of cnn.hip.
// Each returns false, with nothing launched, for a layer it has no build for (the entry point
// then takes the general gather product); otherwise it launches and leaves the status in *err.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dbmp_cnn {

// y = act(conv(x, w) + bias), x [B][H][W][Cin], w [Cout][3][3][Cin]
bool conv_forward_direct(hipStream_t st, const uint16_t *x, int B, int H, int W, int Cin,
                         const uint16_t *w, const float *bias, int Cout, int relu, uint16_t *y,
                         float *y32, hipError_t *err);

// dx = [mask > 0] conv^T(dz, wt), dz [B][H/2][W/2][Cout], wt [Cin][3][3][Cout]
bool conv_backward_data_direct(hipStream_t st, const uint16_t *dz, int B, int H, int W, int Cin,
                               const uint16_t *wt, int Cout, const uint16_t *mask, uint16_t *dx,
                               hipError_t *err);

// dw += dz^T patches(x), db += column sums of dz (db may be null)
bool conv_backward_weight_direct(hipStream_t st, const uint16_t *x, const uint16_t *dz, int B,
                                 int H, int W, int Cin, int Cout, float *dw, float *db,
                                 hipError_t *err);

// The dense layers: y = act(x w^T + bias), x [B][K], w [N][K]
bool linear_forward_direct(hipStream_t st, const uint16_t *x, int B, int K, const uint16_t *w,
                           const float *bias, int N, int relu, uint16_t *y, float *y32,
                           hipError_t *err);

// dx = [mask > 0] dz wt^T, dz [B][N], wt [K][N]
bool linear_backward_data_direct(hipStream_t st, const uint16_t *dz, int B, int N,
                                 const uint16_t *wt, int K, const uint16_t *mask, uint16_t *dx,
                                 hipError_t *err);

// dw += dz^T x, db += column sums of dz (db may be null)
bool linear_backward_weight_direct(hipStream_t st, const uint16_t *x, const uint16_t *dz, int B,
                                   int K, int N, float *dw, float *db, hipError_t *err);

}  // namespace dbmp_cnn
