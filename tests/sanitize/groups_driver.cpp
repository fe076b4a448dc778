// Drives the choice of the groups of interleaved series under AddressSanitizer and UndefinedBehaviorSanitizer without
// a GPU: the launchers are stubs that record what they were given.  Linked like host_driver.cpp.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "rocket_internal.hpp"

static std::string g_route;
static RkGroups g_groups;
static uintptr_t g_copy, g_partial, g_stats;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(&g_route); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { g_route += "mark "; return hipSuccess; }
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

static int backward_short_stub(const rocket_kernels *, const float *, int32_t, const float *, int, int, int, float, float, float,
                               float *, void *) RECORD("backward_short")
static int pad_groups_stub(const rocket_kernels *, const void *, bool is_u8, int32_t, const RkGroups &g, float *xg, void *stats, void *)
{
    g_groups = g;
    g_copy = reinterpret_cast<uintptr_t>(xg);
    g_stats = reinterpret_cast<uintptr_t>(stats);
    g_route += is_u8 ? "pad_groups_u8 " : "pad_groups ";
    return ROCKET_OK;
}
static int backward_groups_stub(const rocket_kernels *, const float *, const RkGroups &, const float *, int, int, int, float, float, float,
                                float *partial, float *, float *, void *)
{
    g_partial = reinterpret_cast<uintptr_t>(partial);
    g_route += "backward_groups ";
    return ROCKET_OK;
}
static int sum_groups_stub(const rocket_kernels *, const RkGroups &, const float *partial, float *, float *, void *)
{
    if (reinterpret_cast<uintptr_t>(partial) == g_partial) g_route += "sum_groups ";
    return ROCKET_OK;
}
static int forward_groups_stub(const rocket_kernels *, const float *, const RkGroups &, uint32_t, float *, void *) RECORD("forward_groups")
static int series_stub(const rocket_kernels *, const float *, int64_t, int32_t, uint32_t, float, float, float *, void *) RECORD("series")
static int forward_wide_stub(const rocket_kernels *, const float *, int32_t, uint32_t, float, float, float *, void *) RECORD("wide")
[[maybe_unused]] static const bool kEntered = (rk_launchers().backward_short = backward_short_stub, rk_launchers().pad_groups = pad_groups_stub,
                                               rk_launchers().backward_groups = backward_groups_stub, rk_launchers().sum_groups = sum_groups_stub,
                                               rk_launchers().forward_groups = forward_groups_stub, rk_launchers().forward_series = series_stub,
                                               rk_launchers().forward_wide = forward_wide_stub, true);

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "check failed at line %d: %s (route: %s, width %d of %d)\n", __LINE__, #cond, g_route.c_str(), g_groups.width, g_groups.first_series); return 1; } } while (0)

alignas(256) static char there[256];

static int backward(rocket_kernels *h, int32_t B, bool u8 = false)
{
    g_route.clear();
    g_groups = rk_groups(B, 1, 1);
    float *at = reinterpret_cast<float *>(there);
    const size_t bytes = rocket_workspace_bytes(h, B, 4, 1);
    return u8 ? rocket_soft_ppv_backward_u8(h, reinterpret_cast<const uint8_t *>(there), B, 4, at, 10.f, -3.f, 0, at, at, there, bytes, nullptr)
              : rocket_soft_ppv_backward(h, at, B, 4, at, 10.f, -3.f, 0, at, at, there, bytes, nullptr);
}

static int forward(rocket_kernels *h, int32_t B, uint32_t mask, bool u8 = false)
{
    g_route.clear();
    g_groups = rk_groups(B, 1, 1);
    float *at = reinterpret_cast<float *>(there);
    const size_t bytes = rocket_workspace_bytes(h, B, mask, 0);
    return u8 ? rocket_transform_u8(h, reinterpret_cast<const uint8_t *>(there), B, mask, 10.f, -3.f, at, there, bytes, nullptr)
              : rocket_transform(h, at, B, mask, 10.f, -3.f, at, there, bytes, nullptr);
}

// The pairs of a launch, as rk_group_pair deals them out: each once.
static int pairs(int32_t K)
{
    const RkGroups &g = g_groups;
    const int rest = g.count % kXcds;
    std::vector<char> seen(static_cast<size_t>(g.count) * K);
    CHECK(g.chunk >= kXcds && g.chunk % kXcds == 0);
    for (int i = 0; i < g.count * K; ++i) {
        int jid, group;
        rk_group_pair_at(g, K, i, jid, group);
        CHECK(jid >= 0 && jid < K && group >= 0 && group < g.count);
        CHECK(seen[static_cast<size_t>(group) * K + jid]++ == 0);
        CHECK((i < rest * K) == (group < rest));
        // an XCD has the same few groups all the way through a round
        if (i >= rest * K) CHECK((group - rest) % kXcds == (i - rest * K) % kXcds);
    }
    return 0;
}

// The series of a batch are in one group each, and what the groups need is inside the workspace.
static int inside(rocket_kernels *h, int32_t B, bool is_backward = true)
{
    const RkGroups &g = g_groups;
    int next = 0, slots = 0;
    for (int i = 0; i < g.count; ++i) {
        CHECK(g.series_before(i) == next && g.slots_before(i) == slots);
        CHECK(g.series_of(i) >= 1 && g.series_of(i) <= g.width_of(i) && g.width_of(i) <= g.width && g.width <= RkGroups::kWidest);
        CHECK(g.width_of(i) >= 2);      // the kernels take a group's dilations to be even
        next += g.series_of(i);
        slots += g.width_of(i);
    }
    CHECK(next == B);
    if (!is_backward) {
        const uintptr_t from = reinterpret_cast<uintptr_t>(there), stats = g_stats;
        CHECK(g_copy == from && from + rk_groups_floats(g, h->C, h->row_len, h->lead) * 4 + 8192 <= stats);
        CHECK(stats + static_cast<uintptr_t>(B) * h->C * 16 <= from + rocket_workspace_bytes(h, B, 3, 0));
        return 0;
    }
    const uintptr_t first = reinterpret_cast<uintptr_t>(there), end = first + rocket_workspace_bytes(h, B, 4, 1);
    CHECK(g_copy == first && g_partial >= first + rk_groups_floats(g, h->C, h->row_len, h->lead) * 4 + 8192);
    const uintptr_t sums = g.count > 1 ? (h->w_off[h->K] + h->K) * 4 * g.count : 0;
    CHECK(g_partial + sums <= g_stats && g_stats + static_cast<uintptr_t>(B) * h->C * 16 <= end);
    return 0;
}

int main()
{
    // the widths that tests/test_gpu_groups.py relies on, then the edges of the rule: one series, few kernels, long series, more tiles
    const struct { int32_t B, C, L, K, width, first; } want[] = {
        {9, 2, 2000, 4000, 2, 1}, {13, 3, 700, 3000, 4, 1}, {27, 2, 400, 2500, 8, 3}, {13, 2, 128, 6000, 16, 13}, {70, 1, 100, 4000, 32, 6},
    {200, 1, 40, 6000, 64, 8}, {130, 1, 25, 4000, 64, 2}, {3, 1, 61, 9000, 4, 3}, {200, 9, 90, 700, 16, 8}, {6, 1, 11, 3000, 8, 6},
        {1, 5, 300, 4000, 1, 1}, {16, 3, 4099, 500, 1, 1}, {64, 20, 17000, 300, 1, 1},
        // too few jobs, or pairs that fill an XCD's L2: slower in groups by 4 to 21 %
        {10, 16, 5462, 2322, 1, 1}, {8, 13, 1339, 1525, 1, 1}, {13, 9, 5401, 2697, 1, 1}, {3, 1, 4321, 8631, 1, 1}, {68, 20, 29054, 4400, 1, 1},
        {80, 17, 29172, 3772, 1, 1}, {60, 20, 32700, 10000, 1, 1},
        // long series that are faster in groups
        {60, 1, 12000, 1000, 2, 2}, {256, 1, 20000, 10000, 8, 8}, {60, 20, 12000, 10000, 2, 2}};
    for (const auto &w : want) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(3, w.K, w.C, w.L, &h) == ROCKET_OK);
        CHECK(backward(h, w.B) == ROCKET_OK);
        CHECK(g_groups.width == w.width && (w.width == 1 || g_groups.first_series == w.first));
        const std::string sum = g_groups.count > 1 ? "sum_groups " : "";       // a single group's sums are the gradients
        CHECK((g_route == "pad_groups backward_groups " + sum) == (w.width > 1));
        if (w.width > 1) {
            if (inside(h, w.B)) return 1;
            CHECK(backward(h, w.B, true) == ROCKET_OK && g_route == "pad_groups_u8 backward_groups " + sum);
            if (inside(h, w.B) || pairs(w.K)) return 1;
            // the timed kernel is the backward kernel, without the sum over the groups
            CHECK(rocket_profile_enable(h, 1) == ROCKET_OK && backward(h, w.B) == ROCKET_OK);
            CHECK(g_route == "pad_groups mark backward_groups mark " + sum);
        }
        rocket_free_kernels(h);
    }
    // one wavefront to a kernel, and four, of tests/test_gpu_backward.py
    const std::string narrow = "pad backward_short reduce ", wide = "pad backward reduce ";
    const struct { int32_t seed, B, C, L, K; std::string route; } alone[] = {
        {1500, 2, 1, 1500, 900, narrow}, {1500, 1, 1, 1500, 900, wide}, {3001, 6, 3, 3001, 900, narrow}, {3001, 3, 3, 3001, 900, wide},
        {8192, 12, 2, 8192, 900, narrow}, {8192, 6, 2, 8192, 900, wide}, {2003, 6, 3, 8192, 4000, narrow}, {2003, 6, 3, 8200, 4000, wide},
        {2003, 6, 3, 8192, 12000, "pad_groups backward_groups sum_groups "}};
    for (const auto &w : alone) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(w.seed, w.K, w.C, w.L, &h) == ROCKET_OK && backward(h, w.B) == ROCKET_OK && g_route == w.route);
        rocket_free_kernels(h);
    }
    // transforms: max and PPV in groups, sums of sigmoids and one-channel sets not
    const struct { int32_t B, C, L, K, width, first; } ahead[] = {
        {28, 15, 134, 2351, 8, 4}, {149, 3, 166, 3236, 32, 21}, {3, 2, 200, 9000, 4, 3}, {149, 18, 1263, 4822, 8, 5}, {9, 4, 600, 6000, 4, 1},
        {130, 2, 60, 4000, 64, 2}, {1, 5, 300, 4000, 1, 1}, {16, 3, 4099, 500, 1, 1}, {64, 5, 8193, 300, 1, 1}};
    for (const auto &w : ahead) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(3, w.K, w.C, w.L, &h) == ROCKET_OK);
        for (uint32_t mask = 1; mask <= 3; ++mask) {
            CHECK(forward(h, w.B, mask) == ROCKET_OK && g_groups.width == w.width && (w.width == 1 || g_groups.first_series == w.first));
            CHECK((g_route == "pad_groups forward_groups ") == (w.width > 1));
            if (w.width == 1) continue;
            if (inside(h, w.B, false) || pairs(w.K)) return 1;
            CHECK(forward(h, w.B, mask, true) == ROCKET_OK && g_route == "pad_groups_u8 forward_groups ");
        }
        CHECK(forward(h, w.B, 7) == ROCKET_OK && g_groups.width == 1);
        rocket_free_kernels(h);
    }
    // four wavefronts to a job where one would be what takes the time; sums of sigmoids stay on one
    const std::string one = "pad short finalize ", four = "pad wide finalize ", group = "pad_groups forward_groups ";
    const struct { int32_t seed, B, C, L, K; std::string route; } width[] = {
        {3, 1, 14, 2857, 1724, four}, {3, 24, 14, 2857, 1724, one}, {3, 24, 20, 8000, 1000, four}, {3, 8, 2, 3000, 2000, one}, {3, 1, 20, 1200, 10000, one},
        {3, 1, 20, 8193, 1000, "pad forward finalize "}, {3, 4, 19, 269, 1122, one}, {3, 5, 19, 417, 870, one}, {3, 1, 19, 512, 170, one},
        {3, 1, 19, 513, 170, four}, {3, 13, 19, 1018, 170, four},
        // of tests/test_gpu_groups.py: a series alone, and its batch
        {1724, 1, 14, 2857, 1724, four}, {1724, 24, 14, 2857, 1724, one}, {2000, 1, 2, 3000, 2000, four}, {2000, 9, 2, 3000, 2000, one},
        {700, 1, 5, 8192, 700, four}, {700, 40, 5, 8192, 700, one}, {300, 1, 1, 1500, 300, four}, {300, 120, 1, 1500, 300, group},
        {1100, 1, 3, 1030, 1100, four}, {1100, 40, 3, 1030, 1100, group}};
    for (const auto &w : width) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(w.seed, w.K, w.C, w.L, &h) == ROCKET_OK);
        for (uint32_t mask = 1; mask <= 3; ++mask) CHECK(forward(h, w.B, mask) == ROCKET_OK && g_route == w.route);
        for (uint32_t mask = 4; mask <= 7; ++mask) CHECK(forward(h, w.B, mask) == ROCKET_OK && g_route == (w.L > 8192 ? "pad forward finalize " : one));
        rocket_free_kernels(h);
    }
    rocket_kernels *sets = nullptr;
    CHECK(rocket_make_kernels(3, 1000, 1, 500, &sets) == ROCKET_OK && forward(sets, 64, 3) == ROCKET_OK && g_route == "series ");
    rocket_free_kernels(sets);
    // all batches of a few handles, one with hardly any partial results to make room in
    const int32_t handles[][3] = {{1, 1, 3000}, {1, 20, 500}, {7, 3, 64}, {300, 2, 200}, {2000, 1, 333}};
    for (const auto &s : handles) {
        rocket_kernels *h = nullptr;
        CHECK(rocket_make_kernels(4, s[0], s[1], s[2], &h) == ROCKET_OK);
        for (int32_t B = 1; B <= 300; ++B) {
            CHECK(backward(h, B) == ROCKET_OK);
            if (g_groups.width > 1 && inside(h, B)) return 1;
            CHECK(forward(h, B, 3) == ROCKET_OK);
            if (g_groups.width > 1 && (inside(h, B, false) || pairs(s[0]))) return 1;
        }
        rocket_free_kernels(h);
    }
    // an imported kernel wider than its series by far stays out of the groups
    const int32_t length = 11, dilation = 300000000, padding = 1500000000, n_ch = 1, channel = 0;
    const float bias = 0.f, weights[11] = {1.f};
    rocket_kernels *h = nullptr;
    CHECK(rocket_kernels_import(1, 1, 100, &length, &dilation, &padding, &bias, &n_ch, &channel, weights, &h) == ROCKET_OK);
    CHECK(backward(h, 64) == ROCKET_OK && g_route == "pad backward_short reduce ");
    rocket_free_kernels(h);
    std::puts("groups driver: ok");
    return 0;
}
