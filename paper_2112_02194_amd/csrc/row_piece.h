// Rows of a table in pieces of eight elements, one piece per lane, and sums over the lanes that share a row.
#pragma once

#include "als_internal.h"

namespace als {

template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// Reduction over groups of G (2, 4, 8, 16) consecutive lanes, the result in every lane.
template <int G, class F> __device__ __forceinline__ float group_reduce(float x, F &&f) {
    x = f(x, dpp_move<0xB1>(x));                          // lanes xor 1
    if constexpr (G > 2) x = f(x, dpp_move<0x4E>(x));     // lanes xor 2
    if constexpr (G > 4) x = f(x, dpp_move<0x141>(x));    // mirror of 8 lanes: the other four
    if constexpr (G > 8) x = f(x, dpp_move<0x140>(x));    // mirror of 16 lanes: the other eight
    return x;
}

// Eight consecutive elements of a row as stored.
template <bool BF16> struct Piece { float4 v[BF16 ? 1 : 2]; };
template <bool BF16> __device__ __forceinline__ Piece<BF16> piece_load(const void *T, int64_t elem) {
    Piece<BF16> p;
    if constexpr (BF16) {
        p.v[0] = *(const float4 *)((const uint16_t *)T + elem);
    } else {
        p.v[0] = *(const float4 *)((const float *)T + elem);
        p.v[1] = *(const float4 *)((const float *)T + elem + 4);
    }
    return p;
}
template <bool BF16> __device__ __forceinline__ Piece<BF16> piece_zero() {
    Piece<BF16> p;
#pragma unroll
    for (auto &v : p.v) v = make_float4(0.f, 0.f, 0.f, 0.f);
    return p;
}
template <bool BF16> __device__ __forceinline__ void piece_floats(const Piece<BF16> &p, float (&x)[8]) {
    if constexpr (BF16) {
        const uint4 w = __builtin_bit_cast(uint4, p.v[0]);
        const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(u[i] << 16);
            x[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
        }
    } else {
        x[0] = p.v[0].x; x[1] = p.v[0].y; x[2] = p.v[0].z; x[3] = p.v[0].w;
        x[4] = p.v[1].x; x[5] = p.v[1].y; x[6] = p.v[1].z; x[7] = p.v[1].w;
    }
}

}  // namespace als
