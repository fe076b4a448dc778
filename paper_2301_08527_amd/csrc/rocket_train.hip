// ROCKET transform for MI355X (gfx950): the small kernels around a training step through
// softPPV (paper section 3.2 makes the pooling differentiable; section 6 names training the
// kernel weights as the next thing to try).  The heavy parts of a step are the transform and
// the backward kernel; here are the loss gradient of a linear head and the parameter update.
//
//   rk_mse_grad   : G[b][i] = (2/B) (pred_b - y_b) coef[i]  and  loss = (1/B) sum_b (pred_b - y_b)^2
//   rk_sgd_update : w <- w - lr*gw, b <- b - lr*gb on the handle's device parameters, with an
//                   optional re-centring of every (kernel, channel) weight row
#include <hip/hip_runtime.h>

#include "rocket_internal.hpp"

// grid (ceil(p/256), B).  Block (0,0) also writes the loss (B is a batch size: a short loop).
__global__ __launch_bounds__(256) void rk_mse_grad(const double *__restrict__ pred, const float *__restrict__ targets,
                                                   const double *__restrict__ coef, int B, int p,
                                                   float *__restrict__ grad_out, double *__restrict__ loss)
{
    const int b = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    const double r = pred[b] - static_cast<double>(targets[b]);
    if (i < p) grad_out[static_cast<size_t>(b) * p + i] = static_cast<float>((2.0 / B) * r * coef[i]);
    if (loss && blockIdx.x == 0 && b == 0 && threadIdx.x == 0) {
        double s = 0.0;
        for (int q = 0; q < B; ++q) {
            const double e = pred[q] - static_cast<double>(targets[q]);
            s += e * e;
        }
        *loss = s / B;
    }
}

// kUpdateRows threads per kernel, thread c for its row of channel c (and c + kUpdateRows, ... of imported kernels with more channels).
// The rows of a kernel one after the other in one thread were a chain of trips to memory: 27 x 19 x 595 samples, 2,590 kernels
// 40 us, so 5.
constexpr int kUpdateRows = 9;       // sampled kernels have no more channels
constexpr int kUpdateKernels = 28;   // of a workgroup
__global__ __launch_bounds__(kUpdateRows * kUpdateKernels) void rk_sgd_update(RkKernelRec *__restrict__ recs, float *__restrict__ weights,
                                                                              const float *__restrict__ gw, const float *__restrict__ gb,
                                                                              int K, float lr, int recentre)
{
    const int kl = static_cast<int>(threadIdx.x) / kUpdateRows, row0 = static_cast<int>(threadIdx.x) - kl * kUpdateRows;
    const int k = static_cast<int>(blockIdx.x) * kUpdateKernels + kl;
    if (k >= K) return;
    const int len = recs[k].len, nch = recs[k].nch, w_off = recs[k].w_off;
    for (int c = row0; c < nch; c += kUpdateRows) {
        float *row = weights + w_off + c * len;
        const float *g = gw + w_off + c * len;
        float v[11], sum = 0.f;
#pragma unroll
        for (int j = 0; j < 11; ++j) {       // all loads of the row are on their way together
            const int at = min(j, len - 1);
            v[j] = fmaf(-lr, g[at], row[at]);
        }
#pragma unroll
        for (int j = 0; j < 11; ++j) sum += j < len ? v[j] : 0.f;
        const float mean = recentre ? sum / static_cast<float>(len) : 0.f;
#pragma unroll
        for (int j = 0; j < 11; ++j)
            if (j < len) row[j] = recentre ? v[j] - mean : v[j];
    }
    if (row0 == 0) recs[k].bias = fmaf(-lr, gb[k], recs[k].bias);
}

int rk_launch_mse_grad(const double *pred, const float *targets, const double *coef, int32_t B, int32_t p,
                       float *grad_out, double *loss, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    hipLaunchKernelGGL(rk_mse_grad, dim3(static_cast<unsigned>((p + 255) / 256), static_cast<unsigned>(B)), dim3(256), 0,
                       stream, pred, targets, coef, B, p, grad_out, loss);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

int rk_launch_sgd_update(const rocket_kernels *h, const float *gw, const float *gb, float lr, int recentre,
                         void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    hipLaunchKernelGGL(rk_sgd_update, dim3(static_cast<unsigned>((h->K + kUpdateKernels - 1) / kUpdateKernels)),
                       dim3(kUpdateRows * kUpdateKernels), 0, stream, const_cast<RkKernelRec *>(h->d_rec), h->d_weights, gw, gb, h->K, lr, recentre);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}
