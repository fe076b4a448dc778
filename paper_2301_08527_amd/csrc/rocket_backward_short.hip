// ROCKET transform for MI355X (gfx950): soft-PPV backward kernel for short series, one 64-lane wavefront per
// (series, kernel).  A kernel with a thousand outputs has some 60 strips: in a workgroup of 256 lanes one wavefront has
// them all, and on the small-dilation path the other three do the same work for nothing.  Bound by vector-instruction issue.
// 64 x 1 x 1,000, 1,000 kernels: 428 -> 169 us; 64 x 6 x 1,500, 500 kernels: 391 -> 211 us.
#include "rocket_backward_impl.hpp"

static int launch_backward_short(const rocket_kernels *h, const float *xpad, int32_t B, const float *grad_out, int F,
                             int plane_soft, int plane_max, float lambda, float nl, float ns, float *partial,
                             void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int J = static_cast<int>(h->jobs.size());
    const int spread = rk_spread(h, B);     // 64 x 1 x 1,000, 1,000 kernels 191 -> 183 us, 240 x 20 x 8,192, 200 kernels 1,980 -> 1,469
    hipLaunchKernelGGL(rk_backward<64>, dim3(static_cast<unsigned>(B) * static_cast<unsigned>(J)), dim3(64), 0, stream, xpad,
                       static_cast<int>(h->row_len), h->lead, h->L, h->C, h->K, J, h->d_rec, h->d_jobs, h->d_bjob_off,
                       h->d_channels, h->d_weights, grad_out, F, plane_soft, plane_max, lambda, nl, ns, partial,
                       static_cast<int>(h->bjob_off.back()), B, spread);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

[[maybe_unused]] static const bool kEntered = (rk_launchers().backward_short = launch_backward_short, true);
