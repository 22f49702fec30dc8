// What the kernels of the dense transform share: the error rows that are formed where they are multiplied,
// 16-byte accesses at any address, rows that end inside a piece.
#pragma once

#include "gather_common.h"

namespace sar {

typedef float float16_t __attribute__((ext_vector_type(16)));

__device__ inline float bf16_to_f32(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

template <typename T>
__device__ inline T from_f32(float v);
template <>
__device__ inline float from_f32<float>(float v) { return v; }
template <>
__device__ inline bf16_t from_f32<bf16_t>(float v) { return bf16_t{(uint16_t)f32_to_bf16_rne(v)}; }

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// ---- error rows that are never stored ---------------------------------------
//
// Z_p.backward(E_p) of Alg. 2 reads the worker's error E_p twice (dW = X^T E_p, dX = E_p W^T).
// For the attention layer E_p = E_{p->p} + ds (x) a_r: the local block's error, stored compactly
// (one row per touched source), plus a rank-one term per head.  Instead of writing that sum out
// and reading it back twice, the two products can form each 16-byte piece of it where they load
// the operand: piece(i, f..) = E[row of i][f..] (zero where E has no row for i) + ds[i, f/D] a_r[f..],
// in fp32 and rounded to the storage type exactly as a stored E_p would have been.
struct RowsOp {
    const int32_t* rank;   // [n+1]: node i's row of E is rank[i], present iff rank[i+1] > rank[i]; null: row i
    const float* ds;       // [n, H] or null (no rank-one term)
    const float* a_r;      // [H*D]
    int H, D;
    int has_E;             // 0: E has no rows at all (or is null)
};

template <typename T>
__device__ inline uint4 fuse_piece(const uint4& base, float d, const float* ar);
template <>
__device__ inline uint4 fuse_piece<float>(const uint4& base, float d, const float* ar)
{
    return make_uint4(__float_as_uint(fmaf(d, ar[0], __uint_as_float(base.x))),
                      __float_as_uint(fmaf(d, ar[1], __uint_as_float(base.y))),
                      __float_as_uint(fmaf(d, ar[2], __uint_as_float(base.z))),
                      __float_as_uint(fmaf(d, ar[3], __uint_as_float(base.w))));
}
template <>
__device__ inline uint4 fuse_piece<bf16_t>(const uint4& base, float d, const float* ar)
{
    float v[8];
    Vec<bf16_t>::unpack(base, v);
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = fmaf(d, ar[x], v[x]);
    uint4 r;
    r.x = pack2_bf16(v[0], v[1]);
    r.y = pack2_bf16(v[2], v[3]);
    r.z = pack2_bf16(v[4], v[5]);
    r.w = pack2_bf16(v[6], v[7]);
    return r;
}

// Any alignment (gfx950 takes unaligned vector accesses).
struct __attribute__((packed, aligned(2))) U4Any {
    uint32_t x, y, z, w;
};
__device__ inline uint4 load16(const void* p)
{
    const U4Any r = *static_cast<const U4Any*>(p);
    return make_uint4(r.x, r.y, r.z, r.w);
}
__device__ inline void store16(void* p, const uint4& v) { *static_cast<U4Any*>(p) = U4Any{v.x, v.y, v.z, v.w}; }

// The last `rest` values of a 16-byte piece, moved to its front, zeros behind them.
template <typename T>
__device__ inline uint4 front_of_piece(const uint4& v, int rest);
template <>
__device__ inline uint4 front_of_piece<float>(const uint4& v, int rest)
{
    return rest == 3 ? make_uint4(v.y, v.z, v.w, 0u) : rest == 2 ? make_uint4(v.z, v.w, 0u, 0u) : make_uint4(v.w, 0u, 0u, 0u);
}
template <>
__device__ inline uint4 front_of_piece<bf16_t>(const uint4& v, int rest)
{
    // down by 8 - rest halves: whole words first, then half a word
    const int words = (8 - rest) >> 1;
    uint32_t w[5] = {v.x, v.y, v.z, v.w, 0u}, o[4];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const bool shift = s < words;
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = shift ? w[k + 1] : w[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = (rest & 1) ? (w[k] >> 16) | (w[k + 1] << 16) : w[k];
    return make_uint4(o[0], o[1], o[2], o[3]);
}

}  // namespace sar
