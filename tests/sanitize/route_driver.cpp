// Drives the host side of the compute entry points under AddressSanitizer and UndefinedBehaviorSanitizer without a GPU:
// the HIP calls of rocket_api.hip are replaced by host memory and the kernel launchers by stubs that record which of them
// a call reached.  Linked like host_driver.cpp.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "rocket_internal.hpp"

static int g_copies = 0, g_mallocs = 0;
static std::string g_route;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { ++g_mallocs; *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { ++g_copies; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
}

#define RECORD(name) { g_route += name " "; return ROCKET_OK; }
int rk_launch_pad(const rocket_kernels *, const float *, int32_t, float *, void *) RECORD("pad")
int rk_launch_mse_grad(const double *, const float *, const double *, int32_t, int32_t, float *, double *, void *) RECORD("mse")
int rk_launch_sgd_update(const rocket_kernels *, const float *, const float *, float, int, void *) RECORD("sgd")
int rk_launch_pad_u8(const rocket_kernels *, const uint8_t *, int32_t, float *, void *, void *) RECORD("pad_u8")
int rk_launch_forward(const rocket_kernels *, const float *, int32_t, uint32_t, float, float, float *, void *) RECORD("forward")
int rk_launch_forward_short(const rocket_kernels *, const float *, int32_t, uint32_t, float, float, float *, void *) RECORD("short")
int rk_launch_finalize(const rocket_kernels *, const float *, int32_t, uint32_t, float *, void *) RECORD("finalize")
int rk_launch_backward(const rocket_kernels *, const float *, int32_t, const float *, int, int, int, float, float, float,
                       float *, void *) RECORD("backward")
int rk_launch_reduce_jobs(const rocket_kernels *, const float *, const float *, int32_t, const float *, int, int, float *,
                          float *, void *) RECORD("reduce")
int rk_launch_minirocket_outputs(const rocket_kernels *, const float *, const int32_t *, int32_t, int32_t, int64_t, float *,
                                 void *) RECORD("mr_outputs")
int rk_launch_minirocket_select(const rocket_kernels *, const int32_t *, int32_t, int32_t, int64_t, const float *, void *)
    RECORD("mr_select")
int rk_launch_minirocket_clear(const rocket_kernels *, int32_t, int32_t *, void *) RECORD("mr_clear")
extern "C" int rocket_ridge_predict(const float *, int32_t, int32_t, const double *, const double *, double *, void *)
    RECORD("ridge_predict")

static int series_stub(const rocket_kernels *, const float *, int64_t, int32_t, uint32_t, float, float, float *, void *) RECORD("series")
static int backward_short_stub(const rocket_kernels *, const float *, int32_t, const float *, int, int, int, float, float, float,
                               float *, void *) RECORD("backward_short")
static int forward_wide_stub(const rocket_kernels *, const float *, int32_t, uint32_t, float, float, float *, void *) RECORD("wide")
static int pad_groups_stub(const rocket_kernels *, const void *, bool, int32_t, const RkGroups &, float *, void *, void *) RECORD("pad_groups")
static int forward_groups_stub(const rocket_kernels *, const float *, const RkGroups &, uint32_t, float *, void *) RECORD("forward_groups")
static int backward_groups_stub(const rocket_kernels *, const float *, const RkGroups &, const float *, int, int, int, float, float, float,
                                float *, float *, float *, void *) RECORD("backward_groups")
static int sum_groups_stub(const rocket_kernels *, const RkGroups &, const float *, float *, float *, void *) RECORD("sum_groups")
[[maybe_unused]] static const bool kEntered = (rk_launchers().forward_series = series_stub, rk_launchers().backward_short = backward_short_stub,
                                               rk_launchers().forward_wide = forward_wide_stub, rk_launchers().pad_groups = pad_groups_stub,
                                               rk_launchers().forward_groups = forward_groups_stub,
                                               rk_launchers().backward_groups = backward_groups_stub, rk_launchers().sum_groups = sum_groups_stub, true);

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "check failed at line %d: %s (route: %s)\n", __LINE__, #cond, g_route.c_str()); return 1; } } while (0)

// The launches of one rocket_transform call.  The stubs touch no sample, so x and the workspace are addresses only.
static std::string transform_route(rocket_kernels *h, int32_t B, uint32_t mask, float lambda = 10.f)
{
    g_route.clear();
    alignas(256) static char there[256];
    const int rc = rocket_transform(h, reinterpret_cast<const float *>(there), B, mask, lambda, -3.f,
                                    reinterpret_cast<float *>(there), there, static_cast<size_t>(1) << 50, nullptr);
    return rc == ROCKET_OK ? g_route : std::string("error ") + rocket_last_error();
}

// One-channel kernels of one length, padded, with the given dilations.
static rocket_kernels *padded_kernels(int32_t L, const std::vector<int32_t> &dilation)
{
    const int32_t K = static_cast<int32_t>(dilation.size());
    std::vector<int32_t> length(K, 11), padding(K), n_ch(K, 1), channels(K, 0);
    std::vector<float> bias(K, 0.5f), weights(11 * static_cast<size_t>(K), 0.25f);
    for (int32_t k = 0; k < K; ++k) padding[k] = 5 * dilation[k];
    rocket_kernels *h = nullptr;
    rocket_kernels_import(K, 1, L, length.data(), dilation.data(), padding.data(), bias.data(), n_ch.data(), channels.data(),
                          weights.data(), &h);
    return h;
}

// Padded kernels may be wider than their series: an imported dilation has no upper limit but its padding's 32 bits.
static int wide_kernels()
{
    rocket_kernels *h = padded_kernels(100, {1, 7, 300000000, 400000000});
    CHECK(h != nullptr);
    CHECK(transform_route(h, 2, 7) == "pad short finalize ");      // too wide for the LDS planes of the series kernel
    const int32_t narrow = 1;
    rocket_kernels *part = nullptr;
    CHECK(rocket_kernels_subset(h, &narrow, 1, &part) == ROCKET_OK);
    CHECK(transform_route(part, 2, 7) == "pad short finalize ");
    rocket_free_kernels(part);
    rocket_free_kernels(h);
    return 0;
}

// Whether a transform goes over sets follows from the handle (and from lambda's sign), never from the batch, and a pruned handle has its
// parent's path.  So it is with the jobs of masks with softPPV; max and PPV alone are the same numbers however they are gathered and go the
// fastest way: one wavefront to a kernel, four, or groups of series.
static int one_path_for_all_batches()
{
    const std::string sets = "series ", jobs = "pad short finalize ";
    const struct { int32_t C, L, K; std::string route; } want[] = {
        {1, 11, 1, sets}, {1, 1000, 4000, sets}, {1, 1024, 1, sets}, {1, 1025, 1024, jobs}, {1, 1025, 1025, sets},
        {1, 5000, 5000, sets}, {1, 5001, 6000, jobs}, {1, 9000, 9500, "pad forward finalize "}, {2, 1000, 4000, jobs}};
    for (const auto &w : want) {
        rocket_kernels *h = nullptr, *part = nullptr;
        CHECK(rocket_make_kernels(3, w.K, w.C, w.L, &h) == ROCKET_OK);
        const int32_t keep = w.K / 2;
        CHECK(rocket_kernels_subset(h, &keep, 1, &part) == ROCKET_OK);
        for (const int32_t B : {1, 16, 256, 4096}) {
            CHECK(transform_route(h, B, 7) == w.route);
            CHECK(transform_route(part, B, 7) == w.route);
            const std::string hard = transform_route(part, B, 3);
            CHECK(hard == w.route || (w.route == jobs && (hard == "pad wide finalize " || hard == "pad_groups forward_groups ")));
        }
        if (w.route == sets) {
            CHECK(transform_route(h, 16, 7, 0.f) == jobs);      // the sets' edges rest on lambda > 0
            CHECK(transform_route(h, 16, 3, 0.f) == sets);      // which max and PPV know nothing of
        }
        rocket_free_kernels(h);
        rocket_free_kernels(part);
    }
    return 0;
}

// Groups of series in the backward pass where they are the faster way; else one wavefront to a job where that is: short series, and longer ones
// with many jobs for their length and channels.
static int backward_paths()
{
    const std::string one = "pad backward_short reduce ", four = "pad backward reduce ", groups = "pad_groups backward_groups sum_groups ";
    const struct { int32_t B, C, L, K; std::string route; } want[] = {
        {1, 1, 11, 1, one}, {4, 20, 1024, 200, one}, {4, 20, 1400, 200, four}, {64, 20, 1400, 200, groups}, {64, 20, 8192, 200, four},
        {64, 20, 8192, 1000, one}, {64, 20, 8193, 1000, groups}, {16, 20, 8193, 1000, four}, {64, 1, 8192, 200, groups}, {4, 1, 8192, 1000, four},
        {16, 6, 4000, 200, four}, {64, 6, 4000, 200, groups}, {10, 16, 5462, 2322, one}};
    for (const auto &w : want) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(3, w.K, w.C, w.L, &h) == ROCKET_OK);
        g_route.clear();
        alignas(256) static char there[256];
        float *at = reinterpret_cast<float *>(there);
        CHECK(rocket_soft_ppv_backward(h, at, w.B, 4, at, 10.f, -3.f, 0, at, at, there, static_cast<size_t>(1) << 50, nullptr) == ROCKET_OK);
        CHECK(g_route == w.route);
        rocket_free_kernels(h);
    }
    return 0;
}

// The parameters reach the device in one allocation and, up to a megabyte, in one copy, on first use and after they were replaced.
static int uploads()
{
    const struct { int32_t K, C; int copies; } want[] = {{70, 1, 1}, {70, 3, 1}, {20000, 1, 9}, {9000, 9, 7}};
    for (const auto &w : want) {
        const int32_t C = w.C;
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(5, w.K, C, 300, &h) == ROCKET_OK);
        g_copies = g_mallocs = 0;
        transform_route(h, 2, 7);
        CHECK(g_copies == w.copies && g_mallocs == 1);
        transform_route(h, 9, 7);
        CHECK(g_copies == w.copies && g_mallocs == 1);
        CHECK(std::memcmp(h->d_weights, h->weights.data(), h->weights.size() * 4) == 0);
        CHECK(std::memcmp(h->d_channels, h->channels.data(), h->channels.size() * 4) == 0);
        CHECK(std::memcmp(h->d_jobs, h->jobs.data(), h->jobs.size() * sizeof(RkJob)) == 0);
        CHECK(std::memcmp(h->d_bjob_off, h->bjob_off.data(), h->bjob_off.size() * 4) == 0);
        CHECK(std::memcmp(h->d_kjob_off, h->kjob_off.data(), h->kjob_off.size() * 4) == 0);
        CHECK(std::memcmp(h->d_kjob_idx, h->kjob_idx.data(), h->kjob_idx.size() * 4) == 0);
        CHECK(h->sets.empty() == (C > 1));
        CHECK(h->sets.empty() || std::memcmp(h->d_sets, h->sets.data(), h->sets.size() * sizeof(RkSet)) == 0);
        CHECK(h->sets.empty() || std::memcmp(h->d_set_rows, h->set_rows.data(), h->set_rows.size() * 4) == 0);
        for (int32_t k = 0; k < h->K; ++k) CHECK(h->d_rec[k].bias == h->bias[k] && h->d_rec[k].w_off == h->w_off[k] && h->d_rec[k].dil == h->dilation[k]);
        std::vector<float> bias(h->bias);
        bias[3] += 1.f;
        CHECK(rocket_kernels_set_params(h, nullptr, bias.data()) == ROCKET_OK);
        transform_route(h, 2, 7);
        CHECK(g_copies == 2 * w.copies && g_mallocs == 1 && h->d_rec[3].bias == bias[3]);
        rocket_free_kernels(h);
    }
    return 0;
}

int main()
{
    if (wide_kernels() || one_path_for_all_batches() || backward_paths() || uploads()) return 1;
    std::puts("route driver: ok");
    return 0;
}
