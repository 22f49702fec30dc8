// An fp32 value as the exact sum of three bf16 values (linear_split.hip says how products are formed of them, and which
// values have no such sum).
#pragma once

#include "linear_common.h"

// (lambdas with several calls must not become functions: their registers are the kernel's)
#define SAR_INLINE __attribute__((always_inline))

namespace sar {

// Eight values as three times eight bf16 values.
__device__ inline void split8(const float (&v)[8], uint4 (&out)[3])
{
    uint32_t p[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = v[2 * j], b = v[2 * j + 1];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            p[t][j] = pack2_bf16(a, b);
            if (t == 2) break;
            a -= __uint_as_float(p[t][j] << 16);
            b -= __uint_as_float(p[t][j] & 0xffff0000u);
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) out[t] = make_uint4(p[t][0], p[t][1], p[t][2], p[t][3]);
}

// The smallest size met, zeros left out: twice its bits less one (zero: the largest number).
constexpr uint32_t kLowBits = 2u * (17u << 23) - 1;      // of 2^-110
__device__ inline uint32_t lowest(uint32_t low, const uint4& v)
{
    low = min(low, min(2u * v.x - 1u, 2u * v.y - 1u));
    return min(low, min(2u * v.z - 1u, 2u * v.w - 1u));
}
// Before `next` is read: put off to where it is read itself, it keeps the values it is taken from in registers of their own
// (dX of 8 tiles 212 -> 221 registers).
__device__ inline void settle(uint32_t& low, float& next) { asm("" : "+v"(low), "+v"(next)); }

constexpr int kTerm[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};

__device__ inline void multiply_split(const uint4 (&a)[3], const uint4 (&b)[3], float16_t& sum)
{
    sum = float16_t{};
#pragma unroll
    for (int t = 0; t < 6; ++t)
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[kTerm[t][0]]),
                                                      __builtin_bit_cast(bf16x8_t, b[kTerm[t][1]]), sum, 0, 0, 0);
}

// Whether an infinity or a NaN is among the results.
__device__ inline bool not_finite(const float16_t& v)
{
    float zero[2] = {0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r % 2] = fmaf(v[r], 0.f, zero[r % 2]);
    return __builtin_isunordered(zero[0], zero[1]);
}

}  // namespace sar
