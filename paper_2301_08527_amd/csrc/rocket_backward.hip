// ROCKET transform for MI355X (gfx950): launch of the soft-PPV backward kernel on long series, and the sum of its jobs.
#include "rocket_backward_impl.hpp"

constexpr int kReduceThreads = 128;      // >= kBwdMaxTerms + 1: one thread per gradient term of a kernel
constexpr int kReduceSeries = 8;         // series whose loads are in flight together

// One workgroup per kernel; thread t < n_ch*len owns weight-gradient term t, thread n_ch*len the
// bias gradient.  Sums the kernel's job partials over the jobs in tile order and over the series in
// ascending b (a fixed order: results repeat bit for bit), finds per series the first
// position of the largest output across the jobs, and adds the max plane's sub-gradient there.
// A series costs two dependent trips to memory (the position of the maximum, the samples there) and little else:
// eight series make them together (64 x 1 x 1,000, 1,000 kernels: the call without the backward kernel 76 -> 48 us).
__global__ __launch_bounds__(kReduceThreads) void rk_reduce_jobs(const float *__restrict__ partial, int B, int stride,
                                                                 const float *__restrict__ xpad, int row_len, int lead, int C,
                                                                 int K, const RkKernelRec *__restrict__ recs,
                                                                 const int32_t *__restrict__ kjob_off,
                                                                 const int32_t *__restrict__ kjob_idx,
                                                                 const int32_t *__restrict__ bjob_off,
                                                                 const int32_t *__restrict__ channels,
                                                                 const float *__restrict__ grad_out, int F, int plane_max,
                                                                 float *__restrict__ grad_w, float *__restrict__ grad_b)
{
    const int kid = blockIdx.x;
    const RkKernelRec rec = recs[kid];
    const int nterms = rec.nch * rec.len;
    const int t = static_cast<int>(threadIdx.x);
    if (t > nterms) return;
    const bool want_max = plane_max >= 0;
    const int q0 = kjob_off[kid], q1 = kjob_off[kid + 1];
    int chan = 0, tap = 0;
    if (t < nterms) {
        const int c = t / rec.len;
        tap = (t - c * rec.len) * rec.dil;
        chan = channels[rec.ch_off + c];
    }
    float sum = 0.f;
    for (int b0 = 0; b0 < B; b0 += kReduceSeries) {
        const float *row[kReduceSeries];
        float part[kReduceSeries], vmax[kReduceSeries];
        int targ[kReduceSeries];
#pragma unroll
        for (int s = 0; s < kReduceSeries; ++s) {             // series past the last repeat its loads
            row[s] = partial + static_cast<size_t>(min(b0 + s, B - 1)) * stride;
            part[s] = 0.f; vmax[s] = -INFINITY; targ[s] = 0;
        }
        for (int q = q0; q < q1; ++q) {
            const int at = bjob_off[kjob_idx[q]];
#pragma unroll
            for (int s = 0; s < kReduceSeries; ++s) {
                const float *job = row[s] + at;
                part[s] += job[t];                            // term t, or the sum of q at t == nterms
                if (want_max) {
                    const float m = job[nterms + 1];
                    const int a = reinterpret_cast<const int *>(job)[nterms + 2];
                    const bool better = m > vmax[s] || (m == vmax[s] && a < targ[s]);
                    vmax[s] = better ? m : vmax[s];
                    targ[s] = better ? a : targ[s];
                }
            }
        }
        float gx[kReduceSeries];                              // with the max plane's share
        if (want_max) {
            float g[kReduceSeries], xv[kReduceSeries];
#pragma unroll
            for (int s = 0; s < kReduceSeries; ++s) {
                const size_t b = static_cast<size_t>(min(b0 + s, B - 1));
                g[s] = grad_out[b * F * K + static_cast<size_t>(plane_max) * K + kid];
                xv[s] = xpad[(b * C + chan) * row_len + (lead - rec.pad) + targ[s] + tap];
            }
#pragma unroll
            for (int s = 0; s < kReduceSeries; ++s) gx[s] = t < nterms ? fmaf(g[s], xv[s], part[s]) : part[s] + g[s];
        } else {
#pragma unroll
            for (int s = 0; s < kReduceSeries; ++s) gx[s] = part[s];
        }
#pragma unroll
        for (int s = 0; s < kReduceSeries; ++s) sum += b0 + s < B ? gx[s] : 0.f;
    }
    if (t < nterms) grad_w[rec.w_off + t] = sum;
    else grad_b[kid] = sum;
}

// ------------------------------------------------------------------ launchers

int rk_launch_backward(const rocket_kernels *h, const float *xpad, int32_t B, const float *grad_out, int F,
                       int plane_soft, int plane_max, float lambda, float nl, float ns, float *partial,
                       void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int J = static_cast<int>(h->jobs.size());
    const int spread = rk_spread(h, B);
    hipLaunchKernelGGL(rk_backward<kThreads>, dim3(static_cast<unsigned>(B) * static_cast<unsigned>(J)), dim3(kThreads), 0, stream, xpad,
                       static_cast<int>(h->row_len), h->lead, h->L, h->C, h->K, J, h->d_rec, h->d_jobs, h->d_bjob_off,
                       h->d_channels, h->d_weights, grad_out, F, plane_soft, plane_max, lambda, nl, ns, partial,
                       static_cast<int>(h->bjob_off.back()), B, spread);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

int rk_launch_reduce_jobs(const rocket_kernels *h, const float *partial, const float *xpad, int32_t B,
                          const float *grad_out, int F, int plane_max, float *grad_w, float *grad_b, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    hipLaunchKernelGGL(rk_reduce_jobs, dim3(static_cast<unsigned>(h->K)), dim3(kReduceThreads), 0, stream, partial, B,
                       static_cast<int>(h->bjob_off.back()), xpad, static_cast<int>(h->row_len), h->lead, h->C, h->K,
                       h->d_rec, h->d_kjob_off, h->d_kjob_idx, h->d_bjob_off, h->d_channels, grad_out, F, plane_max,
                       grad_w, grad_b);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}
