// Internal declarations shared by the host sampler and the HIP translation units.
#pragma once
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "rocket.h"

// Constants shared by the host planner and the kernels.
#ifndef RK_LDS_ROWS
#define RK_LDS_ROWS 17
#endif
#ifndef RK_LDS_MAXD
#define RK_LDS_MAXD 16
#endif
constexpr int kThreads = 256;                 // lanes of the standard workgroup
constexpr int kLdsRows = RK_LDS_ROWS;         // rows per band in the LDS path
constexpr int kLdsMaxD = RK_LDS_MAXD;         // dilations below this take the LDS path
constexpr int kXcds = 8;                       // accelerator dies (XCDs) of the chip, each with its own L2
constexpr int kFewMinD = 256;                 // few-rows path: smallest dilation ...
constexpr int kFewRowsMax = 24;               // ... and largest number of output rows
#ifndef RK_TILE_POSITIONS
#define RK_TILE_POSITIONS 16384
#endif
constexpr int64_t kTilePositions = RK_TILE_POSITIONS;   // smallest time tile of a forward job, in output positions

// MINIROCKET-style kernel set: groups of kMrSet kernels of length kMrLen (rocket.h)
constexpr int kMrSet = 84;
constexpr int kMrLen = 9;
#ifndef RK_MR_TILE
#define RK_MR_TILE 4864
#endif
#ifndef RK_MR_LINEAR_MAXD
#define RK_MR_LINEAR_MAXD 256
#endif
constexpr int kMrTileFloats = RK_MR_TILE;          // channel-summed samples that one workgroup of the group kernel stages in LDS
constexpr int kMrLinearMaxD = RK_MR_LINEAR_MAXD;   // up to this dilation a tile is a run of consecutive positions
static_assert(kMrTileFloats >= 16 * kMrLinearMaxD && kMrTileFloats >= 9 * 256, "a tile must hold its halo and at least one row of outputs");

// One work item of the group kernel (32 bytes).  mode 0: positions [first, first + count) of the group's
// output, `width` = count rounded up to 64.  mode 1: rows [first, first + rows) x columns [col0, col0 + width)
// of the output viewed as rows of d positions.
struct RkMrJob {
    int32_t group, mode, first, count, col0, width, rows, reserved;
};

// One packed record per kernel as the device code reads it (32 bytes).
struct RkKernelRec {
    int32_t len, dil, pad, nout;
    float bias;
    int32_t nch;
    int32_t ch_off;  // into channels[]
    int32_t w_off;   // into weights[]
};

// One forward work item: rows [row0, row1) of kernel `kernel` (rows of d consecutive
// output positions); 16 bytes.
struct RkJob {
    int32_t kernel;
    int32_t row0, row1;
    int32_t flags;   // bit 0: also owns the partial last row; bit 1: covers the whole kernel
};

// Up to 16 kernels of one dilation for rk_forward_series (64 bytes).  Positions are u = t - padding.
constexpr int kSeriesLdsBytes = 159744;  // LDS of a CU that its workgroups may fill
// Whether a handle's kernels go through the sets is decided when it is made, from its length and its number of kernels, and a
// pruned handle keeps what its parent has: a series' features are the same bits in any batch, a kernel's in any pruned handle.
// Up to kSeriesShort samples always, up to kSeriesMost where there are as many kernels as samples.  Sets against job kernels, max and PPV, 64
// series, in us: 1,000 samples and 200, 500, 1,000, 10,000 kernels 20/20, 29/34, 38/58, 156/496; 1,400: 27/23, 44/41, 56/72,
// 222/624; 2,000: 38/27, 65/47, 89/81, 322/691; 4,000: 91/44, 155/78, 227/134, 780/1,170; 8,000 with 2,000: 924/459.  (Few kernels leave
// most sets part-filled, and the more so the more dilations there are.)
constexpr int kSeriesShort = 1024, kSeriesMost = 5000;
struct RkSet {
    int32_t dil;
    int32_t len;               // longest kernel
    int32_t lo, hi;            // positions that any kernel has, lo rounded down to a multiple of 32
    int32_t in_lo, in_hi;      // positions that all kernels have
    int32_t regs;              // result registers in use: ceil(kernels / 4)
    int32_t reserved;
    int8_t tap[16];            // word 4 g + e of lane group g belongs to this tap ...
    int8_t read[16];           // ... or, where that is -1, reads this tap's samples against zero weights
};

// The series of a batch in groups of `width` (a power of two) that lie interleaved in the padded copy: a row of group g holds sample
// t of its series s at t * width_of(g) + s, zeros in front as in the plain copy (lead * width_of(g) of them); the C rows of a
// group and the groups follow one another.  The first group is the one that may be narrower, so that the zeros in front of a
// row are always enough for the reads past the end of the one before; a series left over has a place without one beside it, since the kernels know
// the small dilations of a group as even ones only (3 x 14 x 178 samples, 1,313 kernels, backward, groups of one and two: 72 us, so 47, one series at a time 53).
#ifdef __HIP__
#define RK_BOTH __host__ __device__
#else
#define RK_BOTH
#endif
struct RkGroups {
    static constexpr int kWidest = 64;     // one series for each lane of a wavefront
    int32_t width, count, first_series, first_width;
    int32_t chunk;         // groups that are worked on together once the first count % kXcds are done (a multiple of kXcds)
    int32_t by_kernel;     // those first ones: kernel by kernel (1) or group by group (0)
    RK_BOTH int width_of(int g) const { return g == 0 ? first_width : width; }
    RK_BOTH int series_of(int g) const { return g == 0 ? first_series : width; }
    RK_BOTH int series_before(int g) const { return g == 0 ? 0 : first_series + (g - 1) * width; }      // in the batch
    RK_BOTH int slots_before(int g) const { return g == 0 ? 0 : first_width + (g - 1) * width; }        // in the copy
};
// `series_bytes`: of one series in the padded copy.  The order of the (kernel, group) pairs (rk_group_pair) keeps what is worked on together in the L2s.
constexpr int64_t kGroupBytesOfL2 = 3 << 20;     // of an XCD's 4 MB
inline RkGroups rk_groups(int32_t B, int32_t width, int64_t series_bytes)
{
    RkGroups g;
    g.width = width;
    g.count = (B + width - 1) / width;
    g.first_series = B - (g.count - 1) * width;
    g.first_width = width < 2 ? 1 : 2;
    while (g.first_width < g.first_series) g.first_width *= 2;
    const int64_t bytes = series_bytes * width;
    const int64_t each = kGroupBytesOfL2 / bytes, all = (g.count + kXcds - 1) / kXcds;     // groups of an XCD
    g.chunk = kXcds * static_cast<int32_t>(each < 1 ? 1 : each < all ? each : all);
    g.by_kernel = g.count % kXcds * bytes <= kGroupBytesOfL2;
    return g;
}
// Workgroup `i` -> (kernel in the order of cost, group).  The hardware deals consecutive workgroups out to the XCDs in turn, so of
// kXcds groups side by side each XCD keeps one, whose samples stay in its L2, while all of them go through the kernels, the
// heaviest first.  As many such rounds at a time as the L2s hold; the groups that are left over come first (the end of a launch should
// be light jobs): where all of them fit one L2 side by side too, otherwise one after the other, each on all XCDs.  149 x 18 x 1,263
// samples, 4,822 kernels, max and PPV, eight series to a group: all groups side by side 1,908 us, so 1,132.
RK_BOTH inline void rk_group_pair_at(const RkGroups &groups, int K, int i, int &jid, int &g)
{
    const int rest = groups.count % kXcds;
    if (i < rest * K) {
        if (groups.by_kernel) {
            // by turns, or an even number of groups would give the narrower first one's short jobs to the same XCDs every time
            jid = i / rest;
            g = (i - jid * rest + jid / kXcds) % rest;
        } else {
            g = i / K;
            jid = i - g * K;
        }
        return;
    }
    i -= rest * K;
    const int from = i / (groups.chunk * K) * groups.chunk;
    i -= from * K;
    const int left = groups.count - rest - from, some = groups.chunk < left ? groups.chunk : left;
    jid = i / some;
    g = rest + from + (i - jid * some);
}
// floats of the interleaved copy: its rows, and the zeros that end the last one
inline int64_t rk_groups_floats(const RkGroups &g, int64_t rows, int64_t row_len, int64_t lead)
{
    return g.slots_before(g.count) * rows * row_len + lead * g.width_of(g.count - 1);
}

struct rocket_kernels {
    int32_t K = 0, C = 0, L = 0;
    std::vector<int32_t> length, dilation, padding, n_ch, channels;
    std::vector<float> bias, weights;
    std::vector<int64_t> ch_off, w_off;

    // plan: forward / backward jobs and padded row geometry
    // forward plan: every kernel's rows cut into time tiles; jobs sorted by time window so
    // that workgroups running together read the same stretch of the series
    std::vector<RkJob> jobs;
    std::vector<int32_t> kjob_off, kjob_idx;   // jobs of kernel k: kjob_idx[kjob_off[k] .. kjob_off[k+1])
    // backward pass: job j owns words [bjob_off[j], bjob_off[j+1]) of a series' row of partial
    // results (its kernel's n_ch*len gradient sums + 4 words)
    std::vector<int32_t> bjob_off;
    int32_t pad_max = 0;     // largest padding of any kernel
    int32_t lead = 0;        // zeros in front of every padded row (multiple of 64)
    int64_t row_len = 0;     // floats per padded row (multiple of 64)
    double conv_fma = 0.0;   // sum_k n_k * n_ch_k * len_k
    double outputs = 0.0;    // sum_k n_k
    int32_t max_terms = 0;   // largest n_ch * length of any kernel

    // one channel and short series: sets of kernels of one dilation (empty where the kernels go through the job kernels), the
    // kernels in their 16 rows (-1: none), words of an LDS plane and the index of sample 0 in it
    std::vector<RkSet> sets;
    std::vector<int32_t> set_rows;
    int32_t set_plane = 0, set_origin = 0;

    // device mirror (allocated on first use on `device`)
    int device = -1;
    void *d_blob = nullptr;
    size_t blob_bytes = 0;
    bool params_dirty = true;    // host parameters are newer than the device mirror
    bool host_stale = false;     // the device mirror was updated in place (training) after the last download
    void *update_stream = nullptr;   // stream of that update
    const RkKernelRec *d_rec = nullptr;
    const RkJob *d_jobs = nullptr;
    const int32_t *d_kjob_off = nullptr;
    const int32_t *d_kjob_idx = nullptr;
    const int32_t *d_bjob_off = nullptr;
    const RkSet *d_sets = nullptr;
    const int32_t *d_set_rows = nullptr;
    const int32_t *d_channels = nullptr;
    float *d_weights = nullptr;

    // MINIROCKET-style handles (rocket_minirocket_kernels): number of groups while the weights are the
    // predetermined set (0 otherwise), work items of the group kernel and their device copy (own allocation,
    // made at the first rocket_minirocket_transform)
    int32_t mr_groups = 0;
    std::vector<RkMrJob> mr_jobs;
    const RkMrJob *d_mr_jobs = nullptr;

    // optional event pairs around the dominant kernel of each call
    bool profile = false;
    std::vector<std::pair<void *, void *>> events;
};

void rk_set_error(const std::string &msg);
int rk_fail(int code, const std::string &msg);

// sampler.cpp: fills the per-kernel arrays of `h` (K, C, L already set)
void rk_sample_kernels(uint64_t seed, rocket_kernels &h);
// sampler.cpp: the MINIROCKET-style kernel set (groups of 84 two-valued kernels; C, L already set) and the
// (training example, rank) draws of the biases
void rk_sample_minirocket(uint64_t seed, int32_t groups, rocket_kernels &h);
void rk_minirocket_draws(uint64_t seed, const rocket_kernels &h, int32_t n_train, std::vector<int32_t> &example,
                         std::vector<int32_t> &rank);
// rocket_minirocket.hip: bias-free outputs of kernels [k0, k0 + count) on their drawn examples into ybuf (rows of
// `stride` floats), and the selection of the drawn order statistic, whose negative becomes the kernel's bias in
// the device records
int rk_launch_minirocket_outputs(const rocket_kernels *h, const float *xpad, const int32_t *example_dev, int32_t k0,
                                 int32_t count, int64_t stride, float *ybuf, void *stream);
int rk_launch_minirocket_select(const rocket_kernels *h, const int32_t *rank_dev, int32_t k0, int32_t count,
                                int64_t stride, const float *ybuf, void *stream);
// rocket_minirocket_forward.hip: the PPV features of a MINIROCKET-style handle, group by group: clears the
// B x K counters (the kernel that counts and the one that makes features of them are in the table below)
int rk_launch_minirocket_clear(const rocket_kernels *h, int32_t B, int32_t *counts, void *stream);
// Launchers that the kernels' translation units enter here when the library is loaded: those of the kernels that are an
// alternative to one called directly below (the matrix-core kernels, the one-wavefront backward pass).  The host code links
// without them.
struct RkLaunchers {
    // rocket_forward_series.hip: the transform of a handle's sets (nl < 0 where the mask has softPPV).  x as below.
    int (*forward_series)(const rocket_kernels *h, const float *x, int64_t row_stride, int32_t B, uint32_t mask, float nl, float ns,
                          float *out, void *stream) = nullptr;
    // rocket_forward.hip: rk_launch_forward, for short series too
    int (*forward_wide)(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns, float *partials,
                        void *stream) = nullptr;
    // rocket_minirocket_forward.hip.  x: rows of L samples that start row_stride floats apart.  Adds every work item's
    // positive counts to `counts`, or, where minirocket_one_pass says so, writes the features to `out`.
    int (*minirocket_forward)(const rocket_kernels *h, const float *x, int64_t row_stride, int32_t B, int32_t *counts, float *out,
                              void *stream) = nullptr;
    // The features of those counts (x again: for the few that the matrix cores cannot take).
    int (*minirocket_features)(const rocket_kernels *h, const float *x, int64_t row_stride, const int32_t *counts, int32_t B, float *out,
                               void *stream) = nullptr;
    bool (*minirocket_one_pass)(const rocket_kernels *h, int32_t B) = nullptr;
    // rk_launch_backward with one wavefront to a workgroup
    int (*backward_short)(const rocket_kernels *h, const float *xpad, int32_t B, const float *grad_out, int F, int plane_soft,
                          int plane_max, float lambda, float nl, float ns, float *partial, void *stream) = nullptr;
    // rocket_prologue.hip: the interleaved padded copy, from floats or (`stats` as in rk_launch_pad_u8) from raw bytes
    int (*pad_groups)(const rocket_kernels *h, const void *x, bool is_u8, int32_t B, const RkGroups &groups, float *xg, void *stats,
                      void *stream) = nullptr;
    // rocket_forward_groups.hip: max and PPV (mask without softPPV) over such a copy, features and all
    int (*forward_groups)(const rocket_kernels *h, const float *xg, const RkGroups &groups, uint32_t mask, float *out, void *stream) = nullptr;
    // rocket_backward_groups.hip: the backward pass over such a copy; several groups leave a row of gradients each in `partial`, a single
    // one its gradients
    int (*backward_groups)(const rocket_kernels *h, const float *xg, const RkGroups &groups, const float *grad_out, int F,
                           int plane_soft, int plane_max, float lambda, float nl, float ns, float *partial, float *grad_w,
                           float *grad_b, void *stream) = nullptr;
    // the sum of those rows
    int (*sum_groups)(const rocket_kernels *h, const RkGroups &groups, const float *partial, float *grad_w, float *grad_b, void *stream) = nullptr;
};
RkLaunchers &rk_launchers();      // rocket_api.hip
// rocket_api.hip: offsets, sets, job plan, padded row geometry; returns ROCKET_OK or an error
enum class RkPath { by_size, sets, jobs };      // of one-channel kernels: by the rule at kSeriesShort, or as another handle has them
int rk_finish_handle(rocket_kernels &h, RkPath path = RkPath::by_size);

// Whether a launch over B series uses the per-XCD series mapping (rk_block_to_pair in
// rocket_device.hpp): while the kXcds padded series that are then in flight together fit in half of
// the 256 MB Infinity Cache.  (Measured at 64 x 20 x 50,000, 10,000 kernels: 1 % faster, 22 % less
// L2 fill traffic; fewer kernels re-use a series less: 74 x 14 x 32,734, 342 kernels 1,319 -> 978 us, 13 x 20 x 50,000, 300 kernels
// 540 -> 358; slower at 8 x 20 x 200,000, whose eight padded series are 192 MB, and for the short-series forward kernel, which does
// not use it.)
inline int rk_spread(const rocket_kernels *h, int32_t B)
{
    const int64_t series_bytes = static_cast<int64_t>(h->C) * h->row_len * 4;
    return (B >= kXcds && kXcds * series_bytes <= (128LL << 20)) ? 1 : 0;
}
// Workgroups of a launch over B series x `items` work items each, as the limit on a launch counts them (whole rounds of XCDs).
inline int64_t rk_grid_groups(int32_t B, int64_t items)
{
    return static_cast<int64_t>((B + kXcds - 1) / kXcds) * kXcds * items;
}

// Kernel launchers (rocket_forward.hip, rocket_backward.hip).  `stream` is a hipStream_t.
// They enqueue and return ROCKET_OK, or ROCKET_EHIP if the launch itself was rejected.
int rk_launch_pad(const rocket_kernels *h, const float *x, int32_t B, float *xpad, void *stream);
// rocket_train.hip: loss gradient of a linear head, and the in-place parameter update of
// the handle's device mirror
int rk_launch_mse_grad(const double *pred, const float *targets, const double *coef, int32_t B, int32_t p,
                       float *grad_out, double *loss, void *stream);
int rk_launch_sgd_update(const rocket_kernels *h, const float *gw, const float *gb, float lr, int recentre,
                         void *stream);
// rocket_prologue.hip: the same copy from 8-bit samples, z-normalising every row on the way;
// `stats` is device scratch of 16 bytes per (series, channel) row
int rk_launch_pad_u8(const rocket_kernels *h, const uint8_t *x, int32_t B, float *xpad, void *stats, void *stream);
// forward kernel: one workgroup per (series, job); writes per-job partial results
// (max, positive count, sigmoid sum: three planes of B*J words) into `partials`
int rk_launch_forward(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns,
                      float *partials, void *stream);
// same kernel with one wavefront per workgroup, for short series
int rk_launch_forward_short(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns,
                            float *partials, void *stream);
// combines the per-job partials of every (series, kernel) into the feature planes
int rk_launch_finalize(const rocket_kernels *h, const float *partials, int32_t B, uint32_t mask, float *out,
                       void *stream);
int rk_launch_backward(const rocket_kernels *h, const float *xpad, int32_t B, const float *grad_out, int F,
                       int plane_soft, int plane_max, float lambda, float nl, float ns, float *partial, void *stream);
// sums the job partials of every kernel over the jobs and the batch, adds the max plane's
// sub-gradient at the first arg-max, writes grad_w and grad_b
int rk_launch_reduce_jobs(const rocket_kernels *h, const float *partial, const float *xpad, int32_t B,
                          const float *grad_out, int F, int plane_max, float *grad_w, float *grad_b, void *stream);
