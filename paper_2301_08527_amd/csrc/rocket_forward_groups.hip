// ROCKET transform for MI355X (gfx950): max and PPV of short series, over groups of interleaved series.
//
// The padded copy holds `width` series of a group interleaved (RkGroups), which is one series of width times the samples on which
// a kernel's dilation is width times as large: the paths of rocket_forward_impl.hpp apply as they are, every column count is a
// multiple of `width`, and a lane meets positions of series tid % width only.  A wavefront takes a (kernel, group), closes
// its reductions over the lanes of a series and writes the features: no partial results.  A largest output and a count of
// positive ones are the same numbers in whatever order positions come, so features depend on neither the width nor the batch;
// a sum of sigmoids would, which is why masks with softPPV go one series at a time.
// Bound: vector-instruction issue; what a pass costs whose strips do not fill the lanes.  Which width: the rules at best_groups and
// forward_way in rocket_api.hip.  Max and PPV, one series at a time and in groups: 28 x 15 x 134 samples, 2,351 kernels 94 -> 37 us; 149 x 3 x 166, 3,236
// kernels 402 -> 88 us; 149 x 18 x 1,263, 4,822 kernels 1,640 -> 1,076 us.
#include "rocket_forward_impl.hpp"

namespace {

constexpr int kGroupLanes = 64;

}  // namespace

template <uint32_t MASK>
__attribute__((amdgpu_waves_per_eu(7)))
__global__ __launch_bounds__(kGroupLanes) void rk_forward_groups(const float *__restrict__ xg, int row_len, int lead, int L, int C, int K,
                                                                 const RkKernelRec *__restrict__ recs, const RkJob *__restrict__ jobs,
                                                                 const int32_t *__restrict__ channels, const float *__restrict__ weights,
                                                                 float *__restrict__ out, RkGroups groups)
{
    constexpr int NT = kGroupLanes, F = __builtin_popcount(MASK);
    __shared__ __attribute__((aligned(16))) float tile[rk_tile_words(NT)];   // 16-byte pieces are written straight into it
    int jid, g;
    rk_group_pair(groups, K, jid, g);
    const RkJob job = jobs[jid];
    const RkKernelRec rec = recs[job.kernel];
    KernelCtx k = rk_make_group_ctx(rec, xg, row_len, lead, L, C, groups, g, channels, weights);
    k.mask = MASK;
    PoolState st;
    st.vmax = -INFINITY;
    st.ssum = 0.f;
    st.cnt = 0;
    const int nout = rec.nout * k.width;
    if (rec.len == 7) rk_forward_body<7, NT, true>(k, nout, job, tile, st);
    else if (rec.len == 9) rk_forward_body<9, NT, true>(k, nout, job, tile, st);
    else rk_forward_body<11, NT, true>(k, nout, job, tile, st);

    float vmax = st.vmax;
    int cnt = st.cnt;
    for (int off = NT / 2; off >= k.width; off >>= 1) {
        vmax = fmaxf(vmax, __shfl_xor(vmax, off));
        cnt += __shfl_xor(cnt, off);
    }
    const int s = static_cast<int>(threadIdx.x);
    if (s >= groups.series_of(g)) return;
    float *o = out + static_cast<size_t>(groups.series_before(g) + s) * F * K + job.kernel;
    if constexpr ((MASK & ROCKET_F_MAX) != 0) { *o = vmax + rec.bias; o += K; }
    if constexpr ((MASK & ROCKET_F_PPV) != 0) *o = static_cast<float>(static_cast<double>(cnt) / static_cast<double>(rec.nout));
}

static int launch_forward_groups(const rocket_kernels *h, const float *xg, const RkGroups &groups, uint32_t mask, float *out, void *stream_ptr)
{
    auto launch = [&](auto mc) {
        hipLaunchKernelGGL(rk_forward_groups<decltype(mc)::value>, dim3(static_cast<unsigned>(groups.count) * static_cast<unsigned>(h->K)),
                           dim3(kGroupLanes), 0, static_cast<hipStream_t>(stream_ptr), xg, static_cast<int>(h->row_len), h->lead, h->L, h->C, h->K,
                           h->d_rec, h->d_jobs, h->d_channels, h->d_weights, out, groups);
    };
    if (mask == ROCKET_F_MAX) launch(std::integral_constant<uint32_t, ROCKET_F_MAX>{});
    else if (mask == ROCKET_F_PPV) launch(std::integral_constant<uint32_t, ROCKET_F_PPV>{});
    else launch(std::integral_constant<uint32_t, ROCKET_F_MAX | ROCKET_F_PPV>{});
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

[[maybe_unused]] static const bool kEntered = (rk_launchers().forward_groups = launch_forward_groups, true);
