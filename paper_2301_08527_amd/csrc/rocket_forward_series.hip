// ROCKET transform for MI355X (gfx950): forward kernel for short univariate series, on the bf16 matrix cores.
//
// With one channel, kernels of equal dilation d read the same samples: with u = t - padding the outputs of kernel k are
//     y_k[u] = bias_k + sum_j w_kj x[u + j d],      -padding_k <= u < n_k - padding_k,
// a matrix product of the kernels' weights with the tap values, 16 kernels x 16 positions to an instruction
// (v_mfma_f32_16x16x32_bf16).  fp32 precision comes from splitting samples and weights exactly into three bf16 parts
// (rocket_limbs.hpp) and adding the six products of parts that count:
//     w1 (x1 + x2 + x3) + w2 (x1 + x2) + w3 x1.
// The 32 inner slots are 16 register words of two bf16 numbers, and each tap has one (RkSet::tap).  LDS holds two
// planes of such words, (x1, x2) and (x1, x3); against them stand (w1, w1) and (w2, w2), and (w3, w1): three
// instructions, whatever the lengths, on operands that are LDS words as they stand.
//
// Sets of up to 16 kernels of one dilation are made on the host (plan_sets).  A workgroup stages whole zero-padded
// series in LDS once, as those two planes, and its wavefronts take one set after the other: no partial results, and from floats
// no padded copy of the batch and one launch for the whole transform (raw bytes are normalised into the padded copy
// first).  Which series come here: the rule at kSeriesShort.  The kernel computes E = -y: its sign bit says
// y > 0 (an exact zero comes out as +0), collected with one v_alignbit per output and counted every 32 outputs (a comparison
// would cost two scalar instructions per output, and a SIMD issues one per four clocks).  Kernel i of a set sits in
// row 4 (i % 4) + i / 4, so that a set of f kernels leaves results in ceil(f / 4) of the four result registers and the
// others are not pooled.
// Bound: vector-instruction issue of the pooling (soft PPV: 25 clk of a SIMD per 64 outputs, max 2, PPV 4, the three
// matrix instructions about 7), LDS reads for max and PPV alone on series of thousands of samples.  Measured against the
// job kernels that took these series before: 256 x 1,000 samples, 10,000 kernels, all features 2.15 -> 0.95 ms, max and PPV
// 1.94 -> 0.59 ms; 64 x 400 samples 439 -> 78 us; 64 x 4,000 samples 1.17 -> 0.78 ms (max and PPV); 16 x 512
// samples, 500 kernels, launch-bound 16.5 -> 10 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rocket_device.hpp"
#include "rocket_limbs.hpp"

namespace {

constexpr int kSerStep = 32;               // positions of a step: two matrix instructions wide
constexpr int kSerBlock = 512;             // positions after which counts and sums are put away: 32 sign bits of a register
constexpr int kSerMost = 32;               // most series of a workgroup

// Samples and weights that go through the split: with these limits the smallest product of parts is 2^-120.  A series with another
// sample, or a kernel with another weight, is computed by plain multiply-adds (ser_plain).
__device__ __forceinline__ bool ser_samples_split(const RkSpan &x) { return x.within<-64, 60>(); }
__device__ __forceinline__ bool ser_weights_split(const RkSpan &w) { return w.within<-32, 60>(); }

// min / sum over each row of 16 lanes (all 16 lanes end up with the result)
template <class F>
__device__ __forceinline__ float ser_row16(float v, F &&f)
{
    auto dpp = [&](auto ctrl) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xF, 0xF, true)); };
    v = f(v, dpp(std::integral_constant<int, 0xB1>{}));     // quad_perm [1,0,3,2]
    v = f(v, dpp(std::integral_constant<int, 0x4E>{}));     // quad_perm [2,3,0,1]
    v = f(v, dpp(std::integral_constant<int, 0x124>{}));    // row_ror:4
    v = f(v, dpp(std::integral_constant<int, 0x128>{}));    // row_ror:8
    return v;
}

struct SerState {
    rk_bf16x8 A[3];                     // weight operands: parts 1, 2, 3
    rk_f4 C;                            // -bias of rows 4 g .. 4 g + 3
    int lo[4], n[4];                    // first position and number of outputs of those rows
    float low[4];                       // smallest E
    float soft[2][4], total[4];         // sums of sigmoids: of the last block of positions (by matrix instruction of a step), of those before
    uint32_t bits[4], count[4];
};

// Byte 4 g + e of a 16-byte table in scalar registers.
__device__ __forceinline__ int ser_byte(const int8_t (&table)[16], int g, int e)
{
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t w;
        __builtin_memcpy(&w, table + 4 * i, 4);
        word = g == i ? w : word;
    }
    return static_cast<int8_t>(word >> (8 * e));
}

// Weight operands of a set: lane (row m = lane % 16, g = lane / 16) holds words 4 g .. 4 g + 3 of its row's kernel.
// Returns the rows (bit m) whose weights the split does not carry.
__device__ __forceinline__ uint32_t ser_weights(SerState &st, const RkSet &set, const int32_t *__restrict__ rows, const RkKernelRec *__restrict__ recs,
                                            const float *__restrict__ weights, int lane)
{
    const int m = lane & 15, g = lane >> 4;
    const int k = rows[m];
    int len = 0;
    const float *w = weights;
    if (k >= 0) { len = recs[k].len; w += recs[k].w_off; }
    auto weight = [&](int j) { return j >= 0 && j < len ? 0.f - w[j] : 0.f; };
    uint32_t r[3][4];
    RkSpan span;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t l[3];
        const float v = weight(ser_byte(set.tap, g, e));
        span.add(v);
        rk_split2(v, v, l);
        r[0][e] = l[0];
        r[1][e] = l[1];
        r[2][e] = (l[2] & 0xFFFFu) | l[0] << 16;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) st.A[p] = rk_frag(r[p][0], r[p][1], r[p][2], r[p][3]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int kk = rows[4 * g + v];
        st.C[v] = 0.f; st.lo[v] = 0; st.n[v] = 0;
        if (kk >= 0) { st.C[v] = 0.f - recs[kk].bias; st.lo[v] = -recs[kk].pad; st.n[v] = recs[kk].nout; }
    }
    const uint64_t lanes = __ballot(!ser_weights_split(span));
    if (lanes == 0u) return 0u;
    return static_cast<uint32_t>(lanes | lanes >> 16 | lanes >> 32 | lanes >> 48) & 0xFFFFu;
}

// A word of LDS at a byte address.  A relaxed atomic load, so that the reads of two neighbouring matrix operands are
// not merged into one instruction: its register pairs would have to be moved apart again.
__device__ __forceinline__ uint32_t ser_word(const uint32_t *planes, uint32_t byte)
{
    return __hip_atomic_load(reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(planes) + byte), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Pools the E of 32 positions from u0 (lane: positions u0 + lane % 16 and 16 on), registers v < NV.
template <int MASK, int NV, bool EDGE>
__device__ __forceinline__ void ser_pool(SerState &st, const rk_f4 (&E)[2], int u0, float sl, float ns, int lane)
{
    rk_static_for<0, NV>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        float e[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            e[u] = E[u][v];
            if (EDGE) {       // +inf leaves the minimum, the sign bits and (lambda > 0) the sum of sigmoids as they are
                const bool ok = static_cast<uint32_t>(u0 + 16 * u + (lane & 15) - st.lo[v]) < static_cast<uint32_t>(st.n[v]);
                e[u] = ok ? e[u] : INFINITY;
            }
        }
        if constexpr ((MASK & ROCKET_F_SOFTPPV) != 0) {
            // Eq. 3: 1/(1+exp(-(lambda*y+shift))) = 1/(1+exp2(E*sl + ns)), sl = lambda*log2(e), ns = -shift*log2(e)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                st.soft[u][v] += __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(fmaf(e[u], sl, ns)));
            }
        }
        if constexpr ((MASK & ROCKET_F_MAX) != 0) st.low[v] = fminf(fminf(st.low[v], e[0]), e[1]);
        if constexpr ((MASK & ROCKET_F_PPV) != 0) {
#pragma unroll
            for (int u = 0; u < 2; ++u) st.bits[v] = __builtin_amdgcn_alignbit(st.bits[v], __builtin_bit_cast(uint32_t, e[u]), 31);
        }
    });
}

// Steps from u0 up to `to` (a whole number of them): two of 32 positions at a time, so that their reads share addresses.  Blocks
// end at multiples of kSerBlock, and steps start at multiples of 32, so that a kernel's sum is taken in the same order in any set:
// chains of 16 additions, as 64 lanes have at a thousand positions, then one of the blocks.  (One chain of all the positions of a
// lane had an rms error of 5.2e-8 and 5.4e-8 in the feature at 1,000 and 2,000 samples, the job kernels 4.9e-8 at both.)
template <int MASK, int NV, bool EDGE>
__device__ __forceinline__ void ser_steps(SerState &st, uint32_t (&at)[2][4], uint32_t step, const uint32_t *planes, int &u0, int to,
                                          float sl, float ns, int lane)
{
    while (u0 < to) {
        const int stop = min(to, (u0 & -kSerBlock) + kSerBlock);
        for (; u0 < stop; u0 += 2 * kSerStep) {
            rk_static_for<0, 2>([&](auto hc) {
                constexpr int half = decltype(hc)::value;
                if (half == 0 || u0 + kSerStep < stop) {    // uniform
                    rk_f4 E[2];
                    rk_bf16x8 S12[2], S13[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        uint32_t p[4], q[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            p[e] = ser_word(planes, at[0][e] + (half * 2 + u) * 64u);
                            q[e] = ser_word(planes, at[1][e] + (half * 2 + u) * 64u);
                        }
                        S12[u] = rk_frag(p[0], p[1], p[2], p[3]);
                        S13[u] = rk_frag(q[0], q[1], q[2], q[3]);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) E[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.A[2], S13[u], st.C, 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u) E[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.A[1], S12[u], E[u], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u) E[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.A[0], S12[u], E[u], 0, 0, 0);
                    ser_pool<MASK, NV, EDGE>(st, E, u0 + half * kSerStep, sl, ns, lane);
                }
            });
#pragma unroll
            for (int e = 0; e < 4; ++e) { at[0][e] += step; at[1][e] += step; }
        }
        if (u0 > stop) {        // the last pair was a half: go back to where it ends
            u0 -= kSerStep;
            const uint32_t half = step / 2;
#pragma unroll
            for (int e = 0; e < 4; ++e) { at[0][e] -= half; at[1][e] -= half; }
        }
        if constexpr ((MASK & ROCKET_F_PPV) != 0) {
#pragma unroll
            for (int v = 0; v < NV; ++v) { st.count[v] += static_cast<uint32_t>(__builtin_popcount(st.bits[v])); st.bits[v] = 0u; }
        }
        if constexpr ((MASK & ROCKET_F_SOFTPPV) != 0) {
            if (u0 % kSerBlock == 0) {      // uniform
#pragma unroll
                for (int v = 0; v < NV; ++v) { st.total[v] += st.soft[0][v] + st.soft[1][v]; st.soft[0][v] = st.soft[1][v] = 0.f; }
            }
        }
    }
}

// One set over one series: planes at word `first` of LDS.
template <int MASK, int NV>
__device__ __forceinline__ void ser_run(SerState &st, const RkSet &set, const uint32_t *planes, int first, int plane, int origin,
                                        float sl, float ns, int lane)
{
    static_assert(kSerBlock == 16 * kSerStep, "two sign bits a step");
    const int m = lane & 15, g = lane >> 4;
#pragma unroll
    for (int v = 0; v < NV; ++v) { st.low[v] = INFINITY; st.soft[0][v] = st.soft[1][v] = st.total[v] = 0.f; st.bits[v] = 0u; st.count[v] = 0u; }
    // LDS byte addresses of this lane's four words at the first step
    uint32_t at[2][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        at[0][e] = 4u * static_cast<uint32_t>(first + set.lo + origin + m + ser_byte(set.read, g, e) * set.dil);
        at[1][e] = at[0][e] + 4u * static_cast<uint32_t>(plane);
    }
    uint32_t step = 8u * kSerStep;
    asm volatile("" : "+v"(step));      // additions of vector registers issue twice as fast as those of a scalar one
    // steps before the first position that all kernels have, the steps between, the steps after
    int u0 = set.lo;
    const int end = set.lo + (set.hi - set.lo + kSerStep - 1) / kSerStep * kSerStep;
    const int inner = min(end, set.lo + (set.in_lo - set.lo + kSerStep - 1) / kSerStep * kSerStep);
    const int outer = max(inner, set.lo + (set.in_hi - set.lo) / kSerStep * kSerStep);
    ser_steps<MASK, NV, true>(st, at, step, planes, u0, inner, sl, ns, lane);
    ser_steps<MASK, NV, false>(st, at, step, planes, u0, outer, sl, ns, lane);
    ser_steps<MASK, NV, true>(st, at, step, planes, u0, end, sl, ns, lane);
}

// Features of the rows in registers v < NV of one series.
template <int MASK, int NV>
__device__ __forceinline__ void ser_write(SerState &st, const int32_t *__restrict__ rows, int K, float *__restrict__ out, int lane)
{
    const int m = lane & 15, g = lane >> 4;
    float low = 0.f, soft = 0.f;
    uint32_t count = 0u;
    int n = 1;
    rk_static_for<0, NV>([&](auto vc) {          // lane m keeps the results of register m
        constexpr int v = decltype(vc)::value;
        if constexpr ((MASK & ROCKET_F_MAX) != 0) { const float r = ser_row16(st.low[v], [](float a, float b) { return fminf(a, b); }); low = m == v ? r : low; }
        if constexpr ((MASK & ROCKET_F_SOFTPPV) != 0) { const float r = ser_row16(st.total[v] + (st.soft[0][v] + st.soft[1][v]), [](float a, float b) { return a + b; }); soft = m == v ? r : soft; }
        if constexpr ((MASK & ROCKET_F_PPV) != 0) {
            const int r = rk_row16_sum_int(static_cast<int>(st.count[v]));
            count = m == v ? static_cast<uint32_t>(r) : count;
        }
        n = m == v ? st.n[v] : n;
    });
    const int k = m < NV ? rows[4 * g + m] : -1;
    if (k < 0) return;
    float *o = out + k;
    if constexpr ((MASK & ROCKET_F_MAX) != 0) { *o = 0.f - low; o += K; }
    if constexpr ((MASK & ROCKET_F_PPV) != 0) { *o = static_cast<float>(static_cast<double>(count) / static_cast<double>(n)); o += K; }
    if constexpr ((MASK & ROCKET_F_SOFTPPV) != 0) *o = soft / static_cast<float>(n);
}

// Kernel k over one series, by multiply-adds and pooling as in the job kernels: for the few numbers that the split does not carry.
template <int MASK>
__device__ __forceinline__ void ser_plain(int k, const RkKernelRec *__restrict__ recs, const float *__restrict__ weights,
                                          const float *__restrict__ row, int L, float sl, float ns, int K, float *__restrict__ out, int lane)
{
    asm volatile("" : "+v"(lane));      // or what depends on it alone is computed before the loops over sets and kept
    const RkKernelRec rec = recs[k];
    const float *w = weights + rec.w_off;
    const float nl = 0.f - sl, shifted = fmaf(rec.bias, nl, ns);
    PoolState st = {-INFINITY, 0.f, 0};
    for (int t = lane; t < rec.nout; t += 64) {
        float z[1] = {0.f};
        for (int j = 0; j < rec.len; ++j) {
            const int64_t i = static_cast<int64_t>(t) - rec.pad + static_cast<int64_t>(j) * rec.dil;
            const float v = i >= 0 && i < L ? row[i] : 0.f;
            z[0] = j == 0 ? w[0] * v : fmaf(w[j], v, z[0]);
        }
        rk_pool<1>(z, MASK, -rec.bias, nl, shifted, st);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        st.vmax = fmaxf(st.vmax, __shfl_xor(st.vmax, off));
        st.ssum += __shfl_xor(st.ssum, off);
        if constexpr (rk_counts_by_lane(MASK)) st.cnt += __shfl_xor(st.cnt, off);
    }
    if (lane != 0) return;       // the first lane has a position in every round, and so the wavefront's count
    float *o = out + k;
    if constexpr ((MASK & ROCKET_F_MAX) != 0) { *o = st.vmax + rec.bias; o += K; }
    if constexpr ((MASK & ROCKET_F_PPV) != 0) { *o = static_cast<float>(static_cast<double>(st.cnt) / static_cast<double>(rec.nout)); o += K; }
    if constexpr ((MASK & ROCKET_F_SOFTPPV) != 0) *o = st.ssum / static_cast<float>(rec.nout);
}

}  // namespace

// grid: one workgroup per (block of sets, block of `some` series); its wavefronts take the block's `per` sets in turn,
// each over all of the series.
template <int MASK>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
void rk_forward_series(const float *__restrict__ x, size_t row_stride, int L, const RkKernelRec *__restrict__ recs,
                       const float *__restrict__ weights, const RkSet *__restrict__ sets, const int32_t *__restrict__ set_rows,
                       int nsets, int per, int blocks, int B, int some, int plane, int origin, float sl, float ns,
                       int K, float *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t planes[];    // per series two planes of `plane` words
    __shared__ uint32_t wave_fits[16];
    const int waves = static_cast<int>(blockDim.x) / 64;
    const int tid = static_cast<int>(threadIdx.x);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int sb = static_cast<int>(blockIdx.x) / blocks, block = static_cast<int>(blockIdx.x) - sb * blocks;
    const int b0 = sb * some, nb = min(some, B - b0);
    RkSpan span;
    for (int s = 0; s < nb; ++s) {
        const float *row = x + static_cast<size_t>(b0 + s) * row_stride;
        for (int u = tid * 4; u < plane; u += waves * 256) {
            float v[4];
            const int i = u - origin;
            if (i >= 0 && i <= L - 4) {      // signed: a series may be shorter than four samples
                const f4u q = *reinterpret_cast<const f4u *>(row + i);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = q[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = i + e >= 0 && i + e < L ? row[i + e] : 0.f;
            }
            rk_u32x4 p, q;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float rest;
                span.add(v[e]);
                p[e] = rk_split_pair(v[e], rest);
                q[e] = (p[e] & 0xFFFFu) | rk_pack_bf16(rest, rest) << 16;
            }
            *reinterpret_cast<rk_u32x4 *>(planes + static_cast<size_t>(s) * 2 * plane + u) = p;
            *reinterpret_cast<rk_u32x4 *>(planes + static_cast<size_t>(s) * 2 * plane + plane + u) = q;
        }
    }
    const bool fits = __ballot(!ser_samples_split(span)) == 0u;
    if (lane == 0) wave_fits[wave] = fits;
    __syncthreads();
    uint32_t odd = 0u;       // bit s: series b0 + s has a sample that the split does not carry
    if (__ballot(wave_fits[lane % waves] == 0u) != 0u) {      // uniform
        for (int s = 0; s < nb; ++s) {
            const float *row = x + static_cast<size_t>(b0 + s) * row_stride;
            RkSpan one;
            for (int i = lane; i < L; i += 64) one.add(row[i]);
            if (__ballot(!ser_samples_split(one)) != 0u) odd |= 1u << s;
        }
    }
    asm volatile("" : "+v"(sl), "+v"(ns));
    const int last = min(nsets, (block + 1) * per);
    for (int i = block * per + wave; i < last; i += waves) {
        const RkSet set = sets[i];
        const int32_t *rows = set_rows + 16 * i;
        SerState st;
        const uint32_t odd_rows = ser_weights(st, set, rows, recs, weights, lane);
        for (int s = 0; s < nb; ++s) {
            const int first = s * 2 * plane;
            float *o = out + static_cast<size_t>(b0 + s) * __builtin_popcount(MASK) * K;
            switch (set.regs) {
            case 1: ser_run<MASK, 1>(st, set, planes, first, plane, origin, sl, ns, lane); ser_write<MASK, 1>(st, rows, K, o, lane); break;
            case 2: ser_run<MASK, 2>(st, set, planes, first, plane, origin, sl, ns, lane); ser_write<MASK, 2>(st, rows, K, o, lane); break;
            case 3: ser_run<MASK, 3>(st, set, planes, first, plane, origin, sl, ns, lane); ser_write<MASK, 3>(st, rows, K, o, lane); break;
            default: ser_run<MASK, 4>(st, set, planes, first, plane, origin, sl, ns, lane); ser_write<MASK, 4>(st, rows, K, o, lane); break;
            }
        }
        if ((odd | odd_rows) == 0u) continue;
        __builtin_amdgcn_s_waitcnt(0);      // the features written above are overwritten, by other lanes
        for (int s = 0; s < nb; ++s) {
            float *o = out + static_cast<size_t>(b0 + s) * __builtin_popcount(MASK) * K;
            for (uint32_t plain = (odd >> s & 1u) != 0u ? 0xFFFFu : odd_rows; plain != 0u; plain &= plain - 1u) {
                const int k = rows[__builtin_ctz(plain)];
                if (k >= 0) ser_plain<MASK>(k, recs, weights, x + static_cast<size_t>(b0 + s) * row_stride, L, sl, ns, K, o, lane);
            }
        }
    }
}

static int launch_forward_series(const rocket_kernels *h, const float *x, int64_t row_stride, int32_t B, uint32_t mask, float nl,
                                 float ns, float *out, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const int nsets = static_cast<int>(h->sets.size());
    // A CU holds 16 of these wavefronts: four workgroups of four while a series takes a quarter of its LDS, then two of
    // eight, then one of sixteen.
    const int bytes = 8 * h->set_plane;
    const int waves = bytes <= kSeriesLdsBytes / 4 ? 4 : bytes <= kSeriesLdsBytes / 2 ? 8 : 16;
    // Several series to a workgroup while LDS holds them and enough wavefronts are left: a set's weight operands then
    // serve all of them.
    const int room = std::max(1, kSeriesLdsBytes / 4 * (waves / 4) / bytes);
    const int64_t tasks = static_cast<int64_t>(nsets) * B;
    const int some = static_cast<int>(std::min<int64_t>({room, kSerMost, B, std::max<int64_t>(1, tasks / 16384)}));
    const int64_t sblocks = (B + some - 1) / some;
    // sets of a workgroup: one, two or four to a wavefront
    const int per = waves * (sblocks * nsets >= 131072 ? 4 : sblocks * nsets >= 65536 ? 2 : 1);
    const int blocks = (nsets + per - 1) / per;
    const int lds = bytes * some;
    auto launch = [&](auto mc) {
        auto *kernel = rk_forward_series<decltype(mc)::value>;
        if (lds > 65536 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(sblocks * blocks)), dim3(64 * waves),
                           static_cast<unsigned>(lds), stream, x, static_cast<size_t>(row_stride), h->L, h->d_rec, h->d_weights,
                           h->d_sets, h->d_set_rows, nsets, per, blocks, B, some, h->set_plane, h->set_origin, -nl, ns, h->K, out);
    };
    switch (mask) {
    case 1: launch(std::integral_constant<int, 1>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    case 3: launch(std::integral_constant<int, 3>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 5: launch(std::integral_constant<int, 5>{}); break;
    case 6: launch(std::integral_constant<int, 6>{}); break;
    default: launch(std::integral_constant<int, 7>{}); break;
    }
    return hipGetLastError() == hipSuccess ? ROCKET_OK : ROCKET_EHIP;
}

[[maybe_unused]] static const bool kEntered = (rk_launchers().forward_series = launch_forward_series, true);
