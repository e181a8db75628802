// X = R L^-1 for fp32 tables with d >= 64, sixteen rows of R at a time: fp32 accuracy on the bf16 matrix cores.
#pragma once

#include "dual_common.h"

namespace als {

// Matrix and rows are cut exactly into three bf16 parts each, x = x0 + x1 + x2 with x0 = upper 16 bits of x and so on, and a
// product keeps the six terms m0 x0, m0 x1, m1 x0, m0 x2, m2 x0, m1 x1 (what is dropped is below the rounding of an fp32
// product).  The matrix core's running sum is not rounded to nearest, so only the six products of one 32-column step are
// summed there, from zero and small terms first; the steps are summed on the vector units.
// The matrix supplies the instruction's rows (output columns), the rows of R its columns.  Row m of block o of pair P stands for
// output column 32 P + 8 (m / 4) + 4 o + m % 4, so that lane (n, q) ends up with the eight consecutive output columns
// 32 P + 8 q .. of row n; depth slot (q, i) of a step stands for input column 32 kb + 8 q + i.
// Every row takes the same operations in the same order wherever it comes through here: alone with the kernel that solved it
// (dual_small.hip) or in a pass over the lists (transform_split_kernel).
template <int D> struct XMatrix {
    static constexpr int NK = D / 32;                // steps of 32 input columns, pairs of blocks of 16 output columns
    static constexpr int BLOCKS = NK * (NK + 1);     // 16 x 32 blocks that meet L^-1 (zero above the diagonal)
    static constexpr int BYTES = 3 * 1024 * BLOCKS;  // per block and part: one operand, 16 bytes a lane
    // block o of pair P, step kb >= P
    static constexpr int block(int P, int o, int kb) { return 2 * P * NK - P * (P - 1) + o * (NK - P) + kb - P; }
    // LDS copy of the matrix from its transpose; all threads of the workgroup, a barrier is the caller's
    static __device__ __forceinline__ void fill(char *lds, const float *__restrict__ LinvT, int thread, int threads) {
        for (int e = thread; e < BLOCKS * 64; e += threads) {
            const int b = e >> 6, m = e & 15, q = e >> 4 & 3;
            int P = 0, first = 0;  // the pair and its first block
            while (P + 1 < NK && b >= first + 2 * (NK - P)) {
                first += 2 * (NK - P);
                ++P;
            }
            const int o = b - first >= NK - P, kb = P + b - first - o * (NK - P);
            const float *src = LinvT + (32 * P + 8 * (m >> 2) + 4 * o + (m & 3)) * D + 32 * kb + 8 * q;
            const float4 u = *(const float4 *)src, v = *(const float4 *)(src + 4);
            bf16x8 part[3];
            cut(u, v, part);
#pragma unroll
            for (int t = 0; t < 3; ++t) *(bf16x8 *)(lds + (3 * b + t) * 1024 + (e & 63) * 16) = part[t];
        }
    }
    static __device__ __forceinline__ void cut(const float4 &u, const float4 &v, bf16x8 (&part)[3]) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = pack_upper(x[2 * e], x[2 * e + 1]);
            part[t] = __builtin_bit_cast(bf16x8, w);
            if (t < 2) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = lower_part(x[e]);
            }
        }
    }
};

// NT tiles of sixteen rows: xp[n][t][kb] is part t of the columns 32 kb + 8 q .. of row lane & 15 of tile n; store(n, P, x) gets
// the columns 32 P + 8 q .. of that row, four in x[0] and four in x[1].
template <int D, int NT, class Store>
__device__ __forceinline__ void x_rows(const char *mat, const bf16x8 (&xp)[NT][3][D / 32], Store &&store) {
    using M = XMatrix<D>;
    const char *at = mat + (threadIdx.x & 63) * 16;
    static_for<0, M::NK>([&](auto pp) {
        constexpr int P = decltype(pp)::value;
        floatx4 acc[NT][2];
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[n][0] = acc[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        static_for<P, M::NK>([&](auto kk) {
            constexpr int kb = decltype(kk)::value;
            bf16x8 m[2][3];
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int t = 0; t < 3; ++t) m[o][t] = *(const bf16x8 *)(at + (3 * M::block(P, o, kb) + t) * 1024);
            floatx4 s[NT][2];
#pragma unroll
            for (int n = 0; n < NT; ++n) s[n][0] = s[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            static_for<0, 6>([&](auto xx) {  // small terms first; the chains of the tiles and block columns side by side
                constexpr int x = decltype(xx)::value;
                constexpr int mt[6] = {1, 2, 0, 1, 0, 0}, rt[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int o = 0; o < 2; ++o)
                        s[n][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m[o][mt[x]], xp[n][rt[x]][kb], s[n][o], 0, 0, 0);
            });
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int o = 0; o < 2; ++o) acc[n][o] += s[n][o];
        });
#pragma unroll
        for (int n = 0; n < NT; ++n) store(n, P, acc[n]);
        __builtin_amdgcn_sched_barrier(0);  // keep the next pair's operand reads from piling up
    });
}

}  // namespace als
