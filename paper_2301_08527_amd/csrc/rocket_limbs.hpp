// fp32 arithmetic on the bf16 matrix cores (gfx950): a float as the sum of three bf16 numbers.
//
// With l0 = bf16(x), l1 = bf16(x - l0), l2 = bf16(x - l0 - l1), rounding to nearest, the differences are exact and
// x = l0 + l1 + l2 exactly (three times 8 significant bits and their signs cover the 24 of a float; below about 1e-30
// the last part runs into bf16's subnormal numbers).  A product of two floats is then nine products of parts, each
// exact in fp32; the six with the largest weights leave out terms below 2^-26 of the product, a quarter of one fp32
// rounding.  v_mfma_f32_16x16x32_bf16 adds 32 such products to an fp32 sum: on random data its results lie
// closer to the exact sum (2.4e-8 of the sum of the magnitudes, rms; largest 1.7e-7) than those of a chain of fp32
// fused multiply-adds (2.7e-8; 1.9e-7).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

typedef float rk_f4 __attribute__((ext_vector_type(4)));
typedef __bf16 rk_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 rk_bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t rk_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t rk_u32x4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));      // four floats at any multiple of 4 bytes

// Whether numbers are zeros or of magnitudes in [2^LO, 2^HI] (NaN is not).  The kernels that split take such numbers only, with
// limits that keep every part and every product of parts clear of overflow and of subnormal numbers, and have another path for the
// rest.  Five integer instructions for two numbers (v_min3 and v_max3 take two at a time).
struct RkSpan {
    uint32_t least = 0xFFFFFFFFu, negative = 0u;       // least: of twice the magnitude's bits, less one (zeros come last)
    int32_t positive = 0;
    __device__ __forceinline__ void add(float x)
    {
        const uint32_t bits = __builtin_bit_cast(uint32_t, x);
        least = min(least, (bits << 1) - 1u);
        positive = max(positive, static_cast<int32_t>(bits));
        negative = max(negative, bits);
    }
    template <int LO, int HI>
    __device__ __forceinline__ bool within() const
    {
        constexpr uint32_t hi = static_cast<uint32_t>(HI + 127) << 23;
        return least >= (static_cast<uint32_t>(LO + 127) << 24) - 1u && positive <= static_cast<int32_t>(hi) && negative <= (0x80000000u | hi);
    }
};

__device__ __forceinline__ rk_bf16x8 rk_frag(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_bit_cast(rk_bf16x8, rk_u32x4{a, b, c, d});
}

// two floats rounded to bf16 in one register (first in the low half): v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t rk_pack_bf16(float a, float b)
{
    const rk_bf16x2 v = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
    return __builtin_bit_cast(uint32_t, v);
}

// The parts of two floats, packed: l[p] = part p of a | part p of b << 16.
__device__ __forceinline__ void rk_split2(float a, float b, uint32_t (&l)[3])
{
    l[0] = rk_pack_bf16(a, b);
    asm("" : "+v"(l[0]));      // or the first of the two is rounded a second time to take it apart
    a -= __builtin_bit_cast(float, l[0] << 16);
    b -= __builtin_bit_cast(float, l[0] & 0xFFFF0000u);
    l[1] = rk_pack_bf16(a, b);
    asm("" : "+v"(l[1]));
    a -= __builtin_bit_cast(float, l[1] << 16);
    b -= __builtin_bit_cast(float, l[1] & 0xFFFF0000u);
    l[2] = rk_pack_bf16(a, b);
}

// First and second part of a float, packed (first in the low half); `rest` is what they leave, exact in bf16.
__device__ __forceinline__ uint32_t rk_split_pair(float x, float &rest)
{
    const float r = x - __builtin_bit_cast(float, rk_pack_bf16(x, x) << 16);
    const uint32_t p = rk_pack_bf16(x, r);
    rest = r - __builtin_bit_cast(float, p & 0xFFFF0000u);
    return p;
}

// Stores the parts of four floats to three planes of bf16 numbers, `plane` numbers apart (8-byte aligned).
__device__ __forceinline__ void rk_store_limbs4(const float (&s)[4], unsigned short *at, int plane)
{
    uint32_t lo[3], hi[3];
    rk_split2(s[0], s[1], lo);
    rk_split2(s[2], s[3], hi);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<rk_u32x2 *>(at + p * plane) = rk_u32x2{lo[p], hi[p]};
}

// Two 16-bit numbers of an LDS array at byte offsets lo and hi, in one register.
__device__ __forceinline__ uint32_t rk_lds_pair(const void *base, uint32_t lo, uint32_t hi)
{
    const char *p = static_cast<const char *>(base);
    return static_cast<uint32_t>(*reinterpret_cast<const unsigned short *>(p + lo)) |
           static_cast<uint32_t>(*reinterpret_cast<const unsigned short *>(p + hi)) << 16;
}

// Sum over each row of 16 lanes (all 16 lanes end up with the row sum).
__device__ __forceinline__ int rk_row16_sum_int(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);    // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);   // row_ror:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);   // row_ror:8
    return v;
}
