// ROCKET transform for MI355X (gfx950): the PPV features of MINIROCKET-style kernels, one group at a time.
//
// The paper's related-work section says of MINIROCKET that its weights take two values from a predetermined
// set, so that the convolution can be done by additions, and that it pools with PPV only (Eq. 1-2).  In this
// build's kernel set (rocket.h) the 84 kernels of a group share dilation d, padding and channel subset and
// differ only in which three of their nine weights are 2 (the other six are -1).  With s[t] the sum of the
// group's channels at (zero-padded) sample t and T_j = s[t + j d], kernel k gives y_k = sum_j w_kj T_j: a matrix
// product of the group's 84 x 9 weights with the 9 x n tap values, taken on the matrix cores
// (v_mfma_f32_16x16x32_bf16: 16 kernels x 16 positions).  The bf16 operands lose nothing: a float is the sum of
// three bf16 numbers (8 significant bits each, the split is exact), the weights are exact in bf16, and
// 9 taps x 3 parts fill 27 of the instruction's 32 inner slots; three more hold the bias, split the same way,
// against a constant 1.  Products are exact and sums are kept in fp32 by the instruction.
//
// The kernel computes E = -(y + bias): its sign bit is set exactly where the output is positive (an exact zero comes
// out as +0 and is not counted).  One v_alignbit per output shifts the sign bits into a register, a population count
// every 32 outputs.  The comparison form (v_cmp, s_bcnt1, s_add) that the first version used needs two scalar
// instructions per output and was bound by the one scalar instruction a SIMD issues per four clocks: 10.8 clk per
// output and wavefront against 6.3 for a quarter of a matrix instruction and one v_alignbit (measured back to back).
// The last inner slot multiplies a large positive constant by 1 at positions that do not exist, which clears
// their sign bits.
//
// rk_mr_forward: one workgroup (four wavefronts) per (series, tile of positions of one group).  The
// channel-summed samples that the tile needs are staged in LDS once, as three planes of bf16 parts: for d <= 256 a
// tile is a run of consecutive positions and LDS holds that run plus 8 d samples; for larger d the positions are
// viewed as rows of d (position = row d + column) and a tile is a block of rows x columns, LDS holding rows + 8 rows
// of it.  Either way tap j of the position at LDS index q is at q + j * stride (stride = d, or the block's width).
// The samples come straight from the batch with bounds checks, so no padded copy is made.  Counts are
// integers and added with atomics: the result does not depend on the order.  Where every group is one tile (short
// series) the workgroup writes the features itself.
// Bound by vector-instruction issue: a matrix instruction keeps its unit busy for 16 of a SIMD's clocks and takes some nine of them from
// the others (four wavefronts, 0, 2, 4, 8 and 12 independent multiply-adds to each: 18.5, 19.5, 26.6, 44.0 and 60.5 clk, the multiply-adds
// alone 18.4 for 4, 34.8 for 8, 50.8 for 12), and there are six to seven others to each (84 v_alignbit per 64 positions and lane group, the staging).  Measured at 64 x 20 x 50,000 with 119 groups: 2.57 ms for the call with additions
// and comparisons, 1.97 with the matrix cores, 1.99 with the limits of the split looked after; at 256 x 1 x 1,000
// (rk_mr_forward_series) 258, 175 and 176 us.
// The split carries sums and biases that are zero or in [2^-96, 2^60] in magnitude.  Staging notes others, and such a group of a
// series is counted by plain multiply-adds, where its features are written: the loop over the positions knows nothing of it.
// rk_mr_features: PPV = count / n per (series, kernel).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rocket_internal.hpp"
#include "rocket_device.hpp"
#include "rocket_limbs.hpp"

namespace {

// Tap sets of the 84 kernels: bit j says that weight j is 2.
struct MrSets {
    uint32_t taps[kMrSet];
};
constexpr MrSets mr_sets()
{
    MrSets s{};
    int k = 0;
    for (int a = 0; a < kMrLen; ++a)
        for (int b = a + 1; b < kMrLen; ++b)
            for (int c = b + 1; c < kMrLen; ++c, ++k) s.taps[k] = 1u << a | 1u << b | 1u << c;
    return s;
}

constexpr int kMrTiles = 6;                        // 16-kernel tiles: five full ones and the last four kernels
constexpr int kMrPlane = kMrTileFloats;            // words of a plane
constexpr int kMrMaxPer = 4;                       // most work items of a workgroup
constexpr int kMrChunk = 64;                       // positions a wavefront takes at a time: four matrix instructions wide
// Sums of channels and biases that go through the split; a group of a series with others is counted by mr_plain.
__device__ __forceinline__ bool mr_splits(const RkSpan &s) { return s.within<-96, 60>(); }
constexpr uint32_t kBf16One = 0x3F80, kBf16MinusTwo = 0xC000, kBf16Huge = 0x7F00;   // 1, -2, 2^127

// Row of 16-kernel tile t -> kernel (-1: none).  Register v of a result holds rows 4 g + v of lane group
// g = lane / 16; the last four kernels sit in rows 0, 4, 8, 12, so that only one of that tile's four registers has
// to be looked at.
__host__ __device__ constexpr int mr_kernel(int t, int row) { return t < kMrTiles - 1 ? 16 * t + row : (row % 4 == 0 ? 80 + row / 4 : -1); }
__host__ __device__ constexpr int mr_regs(int t) { return t < kMrTiles - 1 ? 4 : 1; }

// Weight operands without the biases: lane (row m = lane % 16, g = lane / 16) holds inner slots 8 g .. 8 g + 7 of
// kernel row m, two to a register.  With x = x1 + x2 + x3 the parts of a sample, the registers of the sample operand are
//   g = 0: (x1, x2) of taps 0-3      g = 1: (x1, x2) of taps 4-7      g = 2: x3 of taps (0, 1), (2, 3), (4, 5), (6, 7)
//   g = 3: (x1, x2) of tap 8, (x3 of tap 8, unused), (1, 1) and (1, 0 where the position exists and 1 where not)
// and the ones of g = 3 meet the three parts of the bias, the last slot 2^127.  Weights and bias enter negated.
struct MrFrags {
    uint32_t r[kMrTiles][64][4];
};
constexpr MrFrags mr_frags()
{
    const MrSets sets = mr_sets();
    MrFrags f{};
    for (int t = 0; t < kMrTiles; ++t)
        for (int lane = 0; lane < 64; ++lane) {
            const int kk = mr_kernel(t, lane & 15), g = lane >> 4;
            if (kk < 0) continue;
            uint32_t w[kMrLen] = {};
            for (int j = 0; j < kMrLen; ++j) w[j] = (sets.taps[kk] >> j & 1u) ? kBf16MinusTwo : kBf16One;
            for (int e = 0; e < 4; ++e) {
                uint32_t lo = 0, hi = 0;
                if (g < 2) lo = hi = w[4 * g + e];
                else if (g == 2) { lo = w[2 * e]; hi = w[2 * e + 1]; }
                else if (e == 0) lo = hi = w[8];
                else if (e == 1) lo = w[8];
                else if (e == 3) hi = kBf16Huge;
                f.r[t][lane][e] = lo | hi << 16;
            }
        }
    return f;
}
__device__ const MrFrags kFrags = mr_frags();
__device__ const MrSets kTaps = mr_sets();

struct MrState {
    rk_bf16x8 A[kMrTiles];
    uint32_t bits[kMrTiles][4], count[kMrTiles][4];   // sign bits of the last (up to 32) results, positives before them
    int held;                                         // chunks in `bits`
};

template <class F>
__device__ __forceinline__ void mr_each(F &&f)        // every (tile, register) that holds kernels
{
    rk_static_for<0, kMrTiles>([&](auto tc) {
        rk_static_for<0, mr_regs(decltype(tc)::value)>([&](auto vc) { f(tc, vc); });
    });
}

// Weight operands of a group: the table and the biases of its records, which are noted in `span`.
__device__ __forceinline__ void mr_weights(MrState &st, const RkKernelRec *__restrict__ grec, RkSpan &span, int lane)
{
    asm volatile("" : "+v"(lane));      // or the table's entries are loaded before a caller's loop and spilled
    const int m = lane & 15, g = lane >> 4;
    rk_u32x4 r[kMrTiles];
    float bias[kMrTiles];
    rk_static_for<0, kMrTiles>([&](auto tc) {       // all on their way at once: nothing else of a small call is waited for as long
        constexpr int t = decltype(tc)::value;
        const int k = mr_kernel(t, m);
        bias[t] = grec[k < 0 ? 0 : k].bias;
        r[t] = *reinterpret_cast<const rk_u32x4 *>(kFrags.r[t][lane]);
    });
    if (g == 3) {
        rk_static_for<0, kMrTiles / 2>([&](auto hc) {
            constexpr int t = 2 * decltype(hc)::value;
            const float b0 = 0.f - bias[t], b1 = 0.f - bias[t + 1];
            uint32_t l[3];
            rk_split2(b0, b1, l);
            span.add(b0);
            span.add(b1);
            if (mr_kernel(t, m) >= 0) { r[t][2] = (l[0] & 0xFFFFu) | l[1] << 16; r[t][3] |= l[2] & 0xFFFFu; }
            if (mr_kernel(t + 1, m) >= 0) { r[t + 1][2] = l[0] >> 16 | (l[1] & 0xFFFF0000u); r[t + 1][3] |= l[2] >> 16; }
        });
    }
    rk_static_for<0, kMrTiles>([&](auto tc) { st.A[decltype(tc)::value] = __builtin_bit_cast(rk_bf16x8, r[decltype(tc)::value]); });
}
__device__ __forceinline__ void mr_clear(MrState &st)
{
    mr_each([&](auto tc, auto vc) { st.bits[decltype(tc)::value][decltype(vc)::value] = st.count[decltype(tc)::value][decltype(vc)::value] = 0u; });
    st.held = 0;
}
// Moves the sign bits into the counts.
__device__ __forceinline__ void mr_flush(MrState &st)
{
    mr_each([&](auto tc, auto vc) {
        constexpr int t = decltype(tc)::value, v = decltype(vc)::value;
        st.count[t][v] += static_cast<uint32_t>(__builtin_popcount(st.bits[t][v]));
        st.bits[t][v] = 0u;
    });
    st.held = 0;
}

// Where a lane (column lane % 16 = position, g) finds its four registers of the sample operand, as LDS byte addresses
// for the 64 positions from LDS index `first`; registers that are constants stand still when the others move on.
//
// Staged for one stride, every register is one LDS word: kPairs is a plane of words (x1, x2) and a plane of words
// (x3 of q, x3 of q + stride).  Staged for any stride, a register is two 16-bit reads from planes of x1, x2 and x3.
// Behind the planes lie runs of 64 constants.
struct MrPairSlots {        // planes of `plane` words; then runs of the words (1, 1) and (1, 0)
    uint32_t at[4], step, step_hi;
    __device__ __forceinline__ MrPairSlots(int first, int stride, int plane, int positions, int lane)
    {
        const int m = lane & 15, g = lane >> 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int q = first + m;
            if (g < 2) q += (4 * g + e) * stride;
            else if (g == 2) q += plane + 2 * e * stride;
            else if (e < 2) q += e * plane + 8 * stride;
            else q = 2 * plane + (e == 2 ? 0 : kMrChunk);
            at[e] = static_cast<uint32_t>(q) * 4u;
        }
        step = static_cast<uint32_t>(positions) * 4u;
        step_hi = g < 3 ? step : 0u;
    }
    __device__ __forceinline__ void advance() { at[0] += step; at[1] += step; at[2] += step_hi; at[3] += step_hi; }
    __device__ __forceinline__ uint32_t get(const void *planes, int e, uint32_t position) const
    {
        return *reinterpret_cast<const uint32_t *>(static_cast<const char *>(planes) + at[e] + position * 4u);
    }
};
struct MrSingleSlots {      // planes of `plane` 16-bit numbers; then runs of 1 and of 0
    uint32_t lo[4], hi[4], step, step_lo1, step_hi;
    __device__ __forceinline__ MrSingleSlots(int first, int stride, int plane, int positions, int lane)
    {
        const int m = lane & 15, g = lane >> 4, ones = 3 * plane, zeros = ones + kMrChunk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = first + m;
            int a, b;
            if (g < 2) { a = q + (4 * g + e) * stride; b = a + plane; }
            else if (g == 2) { a = q + 2 * plane + 2 * e * stride; b = a + stride; }
            else if (e == 0) { a = q + 8 * stride; b = a + plane; }
            else if (e == 1) { a = q + 2 * plane + 8 * stride; b = zeros; }
            else { a = ones; b = e == 2 ? ones : zeros; }
            lo[e] = static_cast<uint32_t>(a) * 2u;
            hi[e] = static_cast<uint32_t>(b) * 2u;
        }
        step = static_cast<uint32_t>(positions) * 2u;
        step_hi = g < 3 ? step : 0u;
    }
    __device__ __forceinline__ void advance()
    {
        lo[0] += step; hi[0] += step; lo[1] += step; hi[1] += step_hi;
#pragma unroll
        for (int e = 2; e < 4; ++e) { lo[e] += step_hi; hi[e] += step_hi; }
    }
    __device__ __forceinline__ uint32_t get(const void *planes, int e, uint32_t position) const
    {
        return rk_lds_pair(planes, lo[e] + position * 2u, hi[e] + position * 2u);
    }
};

// All 84 kernels at 64 positions, of which the first `valid` exist.
template <class Slots>
__device__ __forceinline__ void mr_chunk(MrState &st, const void *planes, const Slots &slots, int valid, int lane)
{
    const int m = lane & 15, g = lane >> 4;
    uint32_t r[4][4];
    rk_static_for<0, 4>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[u][e] = slots.get(planes, e, 16u * u);
    });
    if (valid < kMrChunk) {     // uniform
        rk_static_for<0, 4>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if (g == 3) r[u][3] = 16 * u + m < valid ? kBf16One : kBf16One << 16 | kBf16One;
        });
    }
    rk_static_for<0, 4>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        const rk_bf16x8 S = rk_frag(r[u][0], r[u][1], r[u][2], r[u][3]);
        rk_static_for<0, kMrTiles>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const rk_f4 E = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.A[t], S, rk_f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            rk_static_for<0, mr_regs(t)>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                const float e = E[v];
                st.bits[t][v] = __builtin_amdgcn_alignbit(st.bits[t][v], __builtin_bit_cast(uint32_t, e), 31);
            });
        });
    });
    if (++st.held == 8) mr_flush(st);       // 32 sign bits per register
}

// Counts of the wavefront, summed over the lanes that share a kernel (two 16-bit counts to a register: a wavefront
// sees fewer than 65,536 positions), to out[kernel], with the sign bit set if `odd`.
__device__ __forceinline__ void mr_counts(MrState &st, int *out, bool odd, int lane)
{
    const int m = lane & 15, g = lane >> 4, sign = odd ? INT32_MIN : 0;
    rk_static_for<0, kMrTiles>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if constexpr (t < kMrTiles - 1) {
            const int a = rk_row16_sum_int(static_cast<int>(st.count[t][0] | st.count[t][1] << 16));
            const int b = rk_row16_sum_int(static_cast<int>(st.count[t][2] | st.count[t][3] << 16));
            if (m < 4) {
                const int c = m < 2 ? a : b;
                out[16 * t + 4 * g + m] = ((m & 1) ? static_cast<int>(static_cast<uint32_t>(c) >> 16) : c & 0xFFFF) | sign;
            }
        } else {
            const int a = rk_row16_sum_int(static_cast<int>(st.count[t][0]));
            if (m == 0) out[80 + g] = a | sign;
        }
    });
}

// Positive outputs of kernel k of a group (record `rec`) over one series, by fp32 multiply-adds on the sums of its channels: for
// what the split does not carry.
__device__ __forceinline__ int mr_plain(const float *series, size_t row_stride, int L, const int32_t *__restrict__ chan, const RkKernelRec &rec,
                                        int k, int lane)
{
    const uint32_t taps = kTaps.taps[k];
    int count = 0;
    for (int t0 = 0; t0 < rec.nout; t0 += 64) {
        float z = 0.f;
#pragma nounroll
        for (int j = 0; j < kMrLen; ++j) {
            const int64_t i = static_cast<int64_t>(t0) + lane - rec.pad + static_cast<int64_t>(j) * rec.dil;
            float s = 0.f;
            if (i >= 0 && i < L) {
#pragma nounroll
                for (int c = 0; c < rec.nch; ++c) {
                    const float v = series[static_cast<size_t>(chan[c]) * row_stride + static_cast<size_t>(i)];
                    s = c == 0 ? v : s + v;
                }
            }
            z = fmaf((taps >> j & 1u) != 0u ? 2.f : -1.f, s, z);
        }
        count += __builtin_popcountll(__ballot(t0 + lane < rec.nout && z > -rec.bias));
    }
    return count;
}

// Fills the LDS planes of a work item with the split sums of the group's NCH channels (added in the order of the
// channel list), noted in `span`.  `series` points at sample 0 of channel 0; index i of the group's view is sample i - pad, 0
// outside [0, L).
template <int NCH>
__device__ __forceinline__ void rk_mr_stage(uint32_t *planes, const float *series, const int32_t *__restrict__ chan,
                                            size_t row_stride, const RkMrJob &job, int d, int stride, int pad, int L, RkSpan &span, int tid)
{
    const float *rows[NCH];
    rk_static_for<0, NCH>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        rows[c] = series + static_cast<size_t>(chan[c]) * row_stride;
    });
    const int total = job.mode == 0 ? job.width + (kMrLen - 1) * d : (job.rows + (kMrLen - 1)) * job.width;
    // four consecutive samples from index i of the view, to LDS index at (a multiple of 4)
    auto four = [&](int i, int at) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        i -= pad;
        if (static_cast<unsigned>(i) <= static_cast<unsigned>(L - 4)) {
            const unsigned byte = static_cast<unsigned>(i) * 4u;    // a 32-bit byte offset beside a scalar row address
            auto load = [&](auto cc) { return *reinterpret_cast<const f4u *>(reinterpret_cast<const char *>(rows[decltype(cc)::value]) + byte); };
            f4u sum = {0.f, 0.f, 0.f, 0.f};
            rk_static_for<0, (NCH + 2) / 3>([&](auto bc) {          // three loads in flight
                constexpr int c0 = 3 * decltype(bc)::value, c1 = c0 + 3 < NCH ? c0 + 3 : NCH;
                f4u v[3];
                rk_static_for<c0, c1>([&](auto cc) { v[decltype(cc)::value - c0] = load(cc); });
                rk_static_for<c0, c1>([&](auto cc) { constexpr int c = decltype(cc)::value; sum = c == 0 ? v[0] : sum + v[c - c0]; });
                __builtin_amdgcn_sched_barrier(0);
            });
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = sum[e];
        } else if (i > -4 && i < L) {
#pragma nounroll
            for (int c = 0; c < NCH; ++c) {
                const float *row = series + static_cast<size_t>(chan[c]) * row_stride;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = i + e >= 0 && i + e < L ? row[i + e] : 0.f;
                    s[e] = c == 0 ? v : s[e] + v;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) span.add(s[e]);
        rk_u32x4 pairs;
        float rest[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) pairs[e] = rk_split_pair(s[e], rest[e]);
        *reinterpret_cast<rk_u32x4 *>(planes + at) = pairs;
        const uint32_t x3[2] = {rk_pack_bf16(rest[0], rest[1]), rk_pack_bf16(rest[2], rest[3])};
        // x3 of a sample is the low half of its own word and the high half of the word `stride` before it
        unsigned short *third = reinterpret_cast<unsigned short *>(planes + kMrPlane + at);
        if (at + 3 + stride < total) {
            rk_static_for<0, 4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                third[2 * e] = static_cast<unsigned short>(x3[e / 2] >> (e & 1) * 16);
            });
        } else {      // nothing lies `stride` after the last ones: their words' high halves must still be numbers
            rk_static_for<0, 4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                const uint32_t v = x3[e / 2] >> (e & 1) * 16 & 0xFFFFu;
                if (at + e + stride < total) third[2 * e] = static_cast<unsigned short>(v);
                else planes[kMrPlane + at + e] = v;
            });
        }
        if (at >= stride) {
            third -= 2 * stride - 1;
            rk_static_for<0, 4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                third[2 * e] = static_cast<unsigned short>(x3[e / 2] >> (e & 1) * 16);
            });
        } else {
            rk_static_for<0, 4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                if (at + e >= stride) third[2 * e - 2 * stride + 1] = static_cast<unsigned short>(x3[e / 2] >> (e & 1) * 16);
            });
        }
    };
    if (job.mode == 0) {
        // positions [first, first + count): LDS index = position - first; filled to where the last lanes read
        for (int u = tid * 4; u < total; u += 1024) four(job.first + u, u);
    } else {
        // output rows [first, first + rows) x columns [col0, col0 + width): LDS index = row * width + column
        const int quads = job.width / 4, row_step = 256 / quads, col_step = 256 - row_step * quads;
        int u = tid / quads, c = tid - u * quads;
        for (; u < job.rows + (kMrLen - 1); u += row_step, c += col_step) {
            if (c >= quads) { c -= quads; ++u; if (u >= job.rows + (kMrLen - 1)) break; }
            four((job.first + u) * d + job.col0 + 4 * c, u * job.width + 4 * c);
        }
    }
}

// grid: workgroups of `per` consecutive work items of a series; mapping as in rk_block_to_pair.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void rk_mr_forward(const float *__restrict__ x, size_t row_stride, int L, int C, const RkKernelRec *__restrict__ recs,
                   const int32_t *__restrict__ channels, const RkMrJob *__restrict__ jobs, int njobs, int per, int B, int spread,
                   int K, int *__restrict__ counts, float *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) uint32_t planes[2 * kMrPlane + 2 * kMrChunk];    // see MrPairSlots
    __shared__ int wave_counts[4][kMrSet];
    int b, block;
    rk_block_to_pair((njobs + per - 1) / per, B, spread, b, block);
    const int tid = static_cast<int>(threadIdx.x);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const float *series = x + static_cast<size_t>(b) * C * row_stride;
    if (tid < 2 * kMrChunk) planes[2 * kMrPlane + tid] = tid < kMrChunk ? kBf16One << 16 | kBf16One : kBf16One;

    MrState st;
    RkSpan span;      // of the group's biases and of the sums that this lane staged
    uint32_t odd_items = 0u;
    const int last = min(njobs, (block + 1) * per);
    for (int item = block * per; item < last; ++item) {
        const RkMrJob job = jobs[item];
        const RkKernelRec *grec = recs + static_cast<size_t>(job.group) * kMrSet;
        const RkKernelRec rec = grec[0];
        const int d = rec.dil, n = rec.nout, nch = rec.nch;
        const int32_t *chan = channels + rec.ch_off;
        if (item == block * per || jobs[item - 1].group != job.group) {
            mr_clear(st);
            span = RkSpan();
            mr_weights(st, grec, span, lane);
        }

        int stride, width, rows, width_valid, limit0, limit_step;
        if (job.mode == 0) {
            stride = d; width = job.width; rows = 1; width_valid = job.count; limit0 = job.count; limit_step = 0;
        } else {
            stride = job.width; width = job.width; rows = job.rows;
            width_valid = min(job.width, d - job.col0);
            limit0 = n - job.first * d - job.col0;     // valid columns of the block's first row if the output ended in it
            limit_step = -d;
        }
        __syncthreads();      // the previous item's planes have been read
        switch (nch) {    // the channel count is a template parameter of the staging loops: loads back to back, no branches
        case 1: rk_mr_stage<1>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 2: rk_mr_stage<2>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 3: rk_mr_stage<3>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 4: rk_mr_stage<4>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 5: rk_mr_stage<5>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 6: rk_mr_stage<6>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 7: rk_mr_stage<7>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        case 8: rk_mr_stage<8>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        default: rk_mr_stage<9>(planes, series, chan, row_stride, job, d, stride, rec.pad, L, span, tid); break;
        }
        MrPairSlots slots(wave * kMrChunk, stride, kMrPlane, 4 * kMrChunk, lane);
        __syncthreads();

        // chunks of 64 columns, dealt to the four wavefronts in turn; `limit0` = valid columns of row 0 and `limit_step`
        // what a row adds to it (rows of the d-column view end where the output ends)
        const int chunks = width / kMrChunk;
        int row = 0, chunk = wave;
        while (chunk >= chunks) { chunk -= chunks; ++row; }
        while (row < rows) {
            const int valid = min(width_valid, limit0 + row * limit_step) - chunk * kMrChunk;
            if (valid > 0) mr_chunk(st, planes, slots, valid, lane);
            slots.advance();
            chunk += 4;
            while (chunk >= chunks) { chunk -= chunks; ++row; }
        }
        mr_flush(st);
        if (item + 1 == last || jobs[item + 1].group != job.group) {
            mr_counts(st, wave_counts[wave], __ballot(!mr_splits(span)) != 0u, lane);
            __syncthreads();
            if (tid < kMrSet) {
                int c[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) c[w] = wave_counts[w][tid];
                const bool odd = (c[0] | c[1] | c[2] | c[3]) < 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) c[w] &= INT32_MAX;
                const int sum = (c[0] + c[1]) + (c[2] + c[3]);
                const size_t to = static_cast<size_t>(b) * K + static_cast<size_t>(job.group) * kMrSet + tid;
                if (out) out[to] = static_cast<float>(static_cast<double>(sum) / static_cast<double>(n));
                else if (odd) atomicOr(counts + to, INT32_MIN);       // a count has no use for the sign bit
                else if (sum != 0) atomicAdd(counts + to, sum);
            }
            if (out && (wave_counts[0][0] | wave_counts[1][0] | wave_counts[2][0] | wave_counts[3][0]) < 0) odd_items |= 1u << (item - block * per);
        }
    }
    if (odd_items != 0u) __syncthreads();      // uniform; the features written above are overwritten
    // features that the split does not carry (those of `counts` are left to rk_mr_features)
    for (uint32_t left = __builtin_amdgcn_readfirstlane(odd_items); left != 0u; left &= left - 1u) {
        const int group = jobs[block * per + __builtin_ctz(left)].group;
        for (int k = wave; k < kMrSet; k += 4) {
            const size_t at = static_cast<size_t>(group) * kMrSet + k;
            const RkKernelRec rec = recs[at];
            const int count = mr_plain(series, row_stride, L, channels + rec.ch_off, rec, k, lane);
            if (lane == 0) out[static_cast<size_t>(b) * K + at] = static_cast<float>(static_cast<double>(count) / static_cast<double>(rec.nout));
        }
    }
}
static_assert(kMrMaxPer <= 32, "a bit for each of a workgroup's items");

// One channel and short series: a workgroup stages its whole zero-padded series once (`pad` zeros on either side) and its
// wavefronts take one group each: nothing is staged per group, and a wavefront that has a group's whole output needs no
// other's counts.  grid: B x `blocks` workgroups, four groups each.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void rk_mr_forward_series(const float *__restrict__ x, size_t row_stride, int L, const RkKernelRec *__restrict__ recs,
                          const int32_t *__restrict__ channels, int groups, int blocks, int pad, int plane, int K, float *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) unsigned short series[];    // 3 planes of `plane` numbers, a run of ones, a run of zeros
    __shared__ int wave_counts[4][kMrSet];
    __shared__ int wave_odd[4];
    const int tid = static_cast<int>(threadIdx.x), b = static_cast<int>(blockIdx.x) / blocks;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = (static_cast<int>(blockIdx.x) - b * blocks) * 4 + wave;
    MrState st;
    mr_clear(st);
    RkSpan bias, span;
    if (g < groups) mr_weights(st, recs + static_cast<size_t>(g) * kMrSet, bias, lane);
    const float *row = x + static_cast<size_t>(b) * row_stride;
    for (int u = tid * 4; u < plane; u += 1024) {
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { const int i = u + e - pad; s[e] = i >= 0 && i < L ? row[i] : 0.f; span.add(s[e]); }
        rk_store_limbs4(s, series + u, plane);
    }
    if (tid < 2 * kMrChunk) series[3 * plane + tid] = tid < kMrChunk ? static_cast<unsigned short>(kBf16One) : static_cast<unsigned short>(0);
    const bool odd_sample = __ballot(!mr_splits(span)) != 0u;
    if (lane == 0) wave_odd[wave] = odd_sample;
    __syncthreads();
    if (g >= groups) return;
    const RkKernelRec rec = recs[static_cast<size_t>(g) * kMrSet];
    MrSingleSlots slots(pad - rec.pad, rec.dil, plane, kMrChunk, lane);
    for (int t = 0; t < rec.nout; t += kMrChunk) {
        mr_chunk(st, series, slots, rec.nout - t, lane);
        slots.advance();
    }
    mr_flush(st);
    mr_counts(st, wave_counts[wave], false, lane);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float *to = out + static_cast<size_t>(b) * K + static_cast<size_t>(g) * kMrSet;
    if (__ballot(!mr_splits(bias)) == 0u && __builtin_amdgcn_readfirstlane(wave_odd[0] | wave_odd[1] | wave_odd[2] | wave_odd[3]) == 0) {
        for (int k = lane; k < kMrSet; k += 64)
            to[k] = static_cast<float>(static_cast<double>(wave_counts[wave][k]) / static_cast<double>(rec.nout));
        return;
    }
    for (int k = 0; k < kMrSet; ++k) {
        const RkKernelRec own = recs[static_cast<size_t>(g) * kMrSet + k];
        const int count = mr_plain(row, row_stride, L, channels + own.ch_off, own, k, lane);
        if (lane == 0) to[k] = static_cast<float>(static_cast<double>(count) / static_cast<double>(own.nout));
    }
}

__global__ __launch_bounds__(256) void rk_mr_clear(int *__restrict__ counts, int total)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < total) counts[i] = 0;
}

// PPV (Eq. 2): the positive count over the kernel's own output length.  Features whose count has the sign bit set are counted
// here, one after the other by a whole wavefront.
__global__ __launch_bounds__(256) void rk_mr_features(const int *__restrict__ counts, int B, int K,
                                                      const RkKernelRec *__restrict__ recs, const float *__restrict__ x, size_t row_stride,
                                                      int L, int C, const int32_t *__restrict__ channels, float *__restrict__ out)
{
    const int i = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
    int count = i < B * K ? counts[i] : 0;
    for (uint64_t left = __ballot(count < 0); left != 0u; left &= left - 1u) {
        const int from = __builtin_ctzll(left), at = i - lane + from;      // uniform
        const int b = at / K, kid = at - b * K;
        const RkKernelRec rec = recs[kid];
        const int found = mr_plain(x + static_cast<size_t>(b) * C * row_stride, row_stride, L, channels + rec.ch_off, rec, kid % kMrSet, lane);
        if (lane == from) count = found;
    }
    if (i >= B * K) return;
    out[i] = static_cast<float>(static_cast<double>(count) / static_cast<double>(recs[i % K].nout));
}

}  // namespace

int rk_launch_minirocket_clear(const rocket_kernels *h, int32_t B, int32_t *counts, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int total = B * h->K;
    hipLaunchKernelGGL(rk_mr_clear, dim3((total + 255) / 256), dim3(256), 0, stream, counts, total);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

// Whether rk_mr_forward_series applies: one channel, and the padded series' planes leave a CU room for four workgroups.
// A wavefront walks over the whole output of its group, so longer series are for batches that fill the chip with groups
// (this kernel against the tiles of rk_mr_forward: 4 x 4,000 samples, 12 groups 47 and 21 us; 64 x 2,000, 40 groups 46 and 40).
static int mr_series_plane(const rocket_kernels *h, int32_t B)
{
    if (h->L > 1024 && static_cast<int64_t>(B) * h->mr_groups < 8192) return 0;
    const int64_t plane = (static_cast<int64_t>(h->L) + 2LL * h->pad_max + kMrChunk + 63) / 64 * 64 + 32;
    return h->C == 1 && plane * 6 <= 39000 ? static_cast<int>(plane) : 0;
}

static bool minirocket_one_pass(const rocket_kernels *h, int32_t B)
{
    return mr_series_plane(h, B) != 0 || h->mr_jobs.size() == static_cast<size_t>(h->mr_groups);
}

static int launch_minirocket_forward(const rocket_kernels *h, const float *x, int64_t row_stride, int32_t B, int32_t *counts,
                                     float *out, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    if (const int plane = mr_series_plane(h, B); plane != 0) {
        const int blocks = (h->mr_groups + 3) / 4;
        hipLaunchKernelGGL(rk_mr_forward_series, dim3(static_cast<unsigned>(static_cast<int64_t>(B) * blocks)), dim3(256),
                           static_cast<unsigned>((3 * plane + 2 * kMrChunk) * 2), stream, x, static_cast<size_t>(row_stride), h->L, h->d_rec,
                           h->d_channels, h->mr_groups, blocks, h->pad_max, plane, h->K, out);
        return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
    }
    const int njobs = static_cast<int>(h->mr_jobs.size());
    const int spread = rk_spread(h, B);
    // items a workgroup takes one after the other (weights and counts stay while they are of one group): as many as
    // leave some eight workgroups for each of a CU's four places
    const int64_t most = static_cast<int64_t>(B) * njobs / 8192;
    const int per = static_cast<int>(most < 1 ? 1 : most > kMrMaxPer ? kMrMaxPer : most);
    const int64_t groups = static_cast<int64_t>(B) * ((njobs + per - 1) / per);
    hipLaunchKernelGGL(rk_mr_forward, dim3(static_cast<unsigned>(groups)), dim3(256), 0, stream, x,
                       static_cast<size_t>(row_stride), h->L, h->C, h->d_rec, h->d_channels, h->d_mr_jobs, njobs, per, B,
                       spread, h->K, counts, out);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

static int launch_minirocket_features(const rocket_kernels *h, const float *x, int64_t row_stride, const int32_t *counts, int32_t B, float *out,
                                      void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int total = B * h->K;
    hipLaunchKernelGGL(rk_mr_features, dim3((total + 255) / 256), dim3(256), 0, stream, counts, B, h->K, h->d_rec, x,
                       static_cast<size_t>(row_stride), h->L, h->C, h->d_channels, out);
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

[[maybe_unused]] static const bool kEntered = (rk_launchers().minirocket_forward = launch_minirocket_forward,
                                               rk_launchers().minirocket_features = launch_minirocket_features,
                                               rk_launchers().minirocket_one_pass = minirocket_one_pass, true);
