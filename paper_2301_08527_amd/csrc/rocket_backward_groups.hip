// ROCKET transform for MI355X (gfx950): soft-PPV backward kernel over groups of short series.
//
// A wavefront that takes one short series has few strips for its 64 lanes (a series of 250 samples has eight strips of 32
// rows) and pays for every kernel and series what a job costs apart from its outputs: the cross-lane sums of n_ch x len
// gradient terms, the remainders of the band heights, the way through descriptors and weights.  `width` series of a group
// (a power of two) therefore lie interleaved in the padded copy, sample t of series s at t * width + s.  That is one series
// of width times the samples, on which the kernel's dilation is width times as large: the strips, bands and loads of
// rocket_backward_impl.hpp apply as they are, every column count is a multiple of `width`, and a lane meets positions of
// one series only, number tid % width.  It has that series' upstream gradient in its coefficient, so the sums over the
// lanes are sums over the group's series at the same time, and one set of partial results is left for each group
// instead of one for each series.  The largest output stays a matter of each series: its position is found over the
// lanes of equal tid % width, and the max plane's sub-gradient is added here, since a job is a whole kernel.
// Bound: vector-instruction issue; few rows to a strip (L / d) and bands that do not fill the lanes are what is left.  Which
// width: the rule at backward_groups in rocket_api.hip.  Whole calls, one series at a time and in groups, the padded copy and the sums
// included: 64 x 1 x 1,000 samples, 1,000 kernels 170 -> 89 us (the kernel alone 80); 28 x 18 x 158, 15,408 kernels 1,695 -> 302 us; 167 x 9 x 1,205,
// 1,737 kernels 1,782 -> 912 us.
#include "rocket_backward_impl.hpp"

namespace {

constexpr int kGroupLanes = 64;
constexpr int kSumThreads = 256;
constexpr int kSumGroups = 8;       // groups whose loads are in flight together

}  // namespace

// grid: one workgroup (one wavefront) per (kernel, group).  xg: the interleaved padded copy.  Writes the kernel's gradient
// sums of the group's series to grad_w + g * stride and grad_b + g * stride.
__global__ __launch_bounds__(kGroupLanes) __attribute__((amdgpu_waves_per_eu(5))) void rk_backward_groups(const float *__restrict__ xg, int row_len, int lead, int L, int C, int K,
                                                                  const RkKernelRec *__restrict__ recs, const RkJob *__restrict__ jobs,
                                                                  const int32_t *__restrict__ channels, const float *__restrict__ weights,
                                                                  const float *__restrict__ grad_out, int F, int plane_soft, int plane_max,
                                                                  float lambda, float nl, float ns, float *__restrict__ grad_w,
                                                                  float *__restrict__ grad_b, size_t stride, RkGroups groups)
{
    constexpr int NT = kGroupLanes, kSlots = rk_bwd_slots(NT);
    __shared__ __attribute__((aligned(16))) float tile[rk_tile_words(NT)];   // 16-byte pieces are written straight into it
    __shared__ float slots[(kBwdMaxTerms + 1) * kSlots];
    __shared__ float s_g[RkGroups::kWidest];
    __shared__ int s_at[RkGroups::kWidest];
    int jid, g;
    rk_group_pair(groups, K, jid, g);
    const RkJob job = jobs[jid];
    const int kid = job.kernel;
    const RkKernelRec rec = recs[kid];
    const int tid = static_cast<int>(threadIdx.x);
    const int width = groups.width_of(g), series = groups.series_of(g);
    const int s = tid & (width - 1);
    KernelCtx k = rk_make_group_ctx(rec, xg, row_len, lead, L, C, groups, g, channels, weights);
    k.nl = nl;
    k.ns = fmaf(rec.bias, nl, ns);

    const int nterms = rec.nch * rec.len;
    for (int i = tid; i < nterms * kSlots; i += NT) slots[i] = 0.f;
    if (tid < kSlots) slots[kBwdMaxTerms * kSlots + tid] = 0.f;
    __syncthreads();

    const bool want_max = plane_max >= 0;
    const float *g_row = grad_out + static_cast<size_t>(groups.series_before(g) + s) * F * K + kid;
    const float coef = s < series ? g_row[static_cast<size_t>(plane_soft) * K] * lambda / static_cast<float>(rec.nout) : 0.f;
    BwdState st;
    st.qsum = 0.f;
    st.vmax = -INFINITY;
    st.targ = s;            // position 0 of the lane's series
    if (rec.len == 7) rk_backward_body<NT, true, 7>(k, rec.nout * width, job, coef, want_max, tile, slots, st);
    else if (rec.len == 9) rk_backward_body<NT, true, 9>(k, rec.nout * width, job, coef, want_max, tile, slots, st);
    else rk_backward_body<NT, true, 11>(k, rec.nout * width, job, coef, want_max, tile, slots, st);

    // (max, first position) of every series: over the lanes that have it
    if (want_max) {
        float vmax = st.vmax;
        int targ = st.targ;
        for (int off = NT / 2; off >= width; off >>= 1) {
            const float om = __shfl_xor(vmax, off);
            const int ot = __shfl_xor(targ, off);
            if (om > vmax || (om == vmax && ot < targ)) { vmax = om; targ = ot; }
        }
        if (tid < width) {
            s_g[tid] = tid < series ? g_row[static_cast<size_t>(plane_max) * K] : 0.f;
            s_at[tid] = targ;
        }
    }
    __syncthreads();        // also orders the slot updates before the slot sums below
    float *gw = grad_w + static_cast<size_t>(g) * stride + rec.w_off;
    for (int t = tid; t < nterms; t += NT) {
        float sum = 0.f;
#pragma unroll
        for (int l = 0; l < kSlots; ++l) sum += slots[t * kSlots + l];
        if (want_max) {
            const int c = t / rec.len;
            const float *x = reinterpret_cast<const float *>(k.xk + static_cast<size_t>(k.chans[c]) * k.row_bytes) + (t - c * rec.len) * k.d;
#pragma unroll 4
            for (int b = 0; b < width; ++b) sum = fmaf(s_g[b], x[s_at[b]], sum);
        }
        gw[t] = sum;
    }
    if (tid == 0) {
        const float *q = slots + kBwdMaxTerms * kSlots;
        float sum = (q[0] + q[1]) + (q[2] + q[3]);
        if (want_max)
            for (int b = 0; b < width; ++b) sum += s_g[b];
        grad_b[static_cast<size_t>(g) * stride + kid] = sum;
    }
}

// Sums the groups' rows of `nw` weight gradients and `nb` bias gradients, in order.
__global__ __launch_bounds__(kSumThreads) void rk_sum_groups(const float *__restrict__ partial, int groups, int nw, int nb,
                                                             float *__restrict__ grad_w, float *__restrict__ grad_b)
{
    const int i = static_cast<int>(blockIdx.x) * kSumThreads + static_cast<int>(threadIdx.x), n = nw + nb;
    if (i >= n) return;
    float sum = 0.f;
    for (int g0 = 0; g0 < groups; g0 += kSumGroups) {
        float v[kSumGroups];
#pragma unroll
        for (int g = 0; g < kSumGroups; ++g) v[g] = partial[static_cast<size_t>(min(g0 + g, groups - 1)) * n + i];
#pragma unroll
        for (int g = 0; g < kSumGroups; ++g) sum += g0 + g < groups ? v[g] : 0.f;
    }
    if (i < nw) grad_w[i] = sum;
    else grad_b[i - nw] = sum;
}

static int launch_backward_groups(const rocket_kernels *h, const float *xg, const RkGroups &groups, const float *grad_out, int F,
                                  int plane_soft, int plane_max, float lambda, float nl, float ns, float *partial, float *grad_w,
                                  float *grad_b, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int nw = static_cast<int>(h->w_off[h->K]);
    const bool direct = groups.count == 1;      // no partial results
    hipLaunchKernelGGL(rk_backward_groups, dim3(static_cast<unsigned>(groups.count) * static_cast<unsigned>(h->K)), dim3(kGroupLanes), 0,
                       stream, xg, static_cast<int>(h->row_len), h->lead, h->L, h->C, h->K, h->d_rec, h->d_jobs, h->d_channels,
                       h->d_weights, grad_out, F, plane_soft, plane_max, lambda, nl, ns, direct ? grad_w : partial,
                       direct ? grad_b : partial + nw, direct ? 0 : static_cast<size_t>(nw) + h->K, groups);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

static int launch_sum_groups(const rocket_kernels *h, const RkGroups &groups, const float *partial, float *grad_w, float *grad_b, void *stream)
{
    const int nw = static_cast<int>(h->w_off[h->K]);
    hipLaunchKernelGGL(rk_sum_groups, dim3(static_cast<unsigned>((static_cast<int64_t>(nw) + h->K + kSumThreads - 1) / kSumThreads)),
                       dim3(kSumThreads), 0, static_cast<hipStream_t>(stream), partial, groups.count, nw, h->K, grad_w, grad_b);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

[[maybe_unused]] static const bool kEntered = (rk_launchers().backward_groups = launch_backward_groups, rk_launchers().sum_groups = launch_sum_groups,
                                               true);
