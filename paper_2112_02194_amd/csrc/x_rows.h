// X = R L^-1, sixteen rows of R at a time, on the bf16 matrix cores: for fp32 tables (d >= 64) with fp32 accuracy, for bf16 tables
// (d >= 32) with the accuracy of their rounding.
#pragma once

#include "dual_common.h"

namespace als {

__device__ __forceinline__ uint32_t pack_nearest(float x, float y) {  // two bf16, rounded to nearest even
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){x, y}, bf16x2));
}

// fp32: matrix and rows are cut exactly into three bf16 parts each, x = x0 + x1 + x2 with x0 = upper 16 bits of x and so on, and a
// product keeps the six terms m0 x0, m0 x1, m1 x0, m0 x2, m2 x0, m1 x1 (what is dropped is below the rounding of an fp32
// product).  The matrix core's running sum is not rounded to nearest, so only the six products of one 32-column step are
// summed there, from zero and small terms first; the steps are summed on the vector units.
// bf16: two parts each, x = bf16(x) + bf16(x - bf16(x)), and three terms, summed in the matrix core: the error of the cut, 2^-17
// relative, is far below the rounding of the output.
// The matrix supplies the instruction's rows (output columns), the rows of R its columns.  Row m of block o of pair P stands for
// output column 32 P + 8 (m / 4) + 4 o + m % 4, so that lane (n, q) ends up with the eight consecutive output columns
// 32 P + 8 q .. of row n; depth slot (q, i) of a step stands for input column 32 kb + 8 q + i.
// Every row takes the same operations in the same order wherever it comes through here: in the kernel that solved it or in a pass
// over the lists (transform_lists_kernel).
template <int D, bool BF> struct XMatrix {
    static constexpr int PARTS = BF ? 2 : 3;
    static constexpr int NK = D / 32;                // steps of 32 input columns, pairs of blocks of 16 output columns
    static constexpr int BLOCKS = NK * (NK + 1);     // 16 x 32 blocks that meet L^-1 (zero above the diagonal)
    static constexpr int BYTES = PARTS * 1024 * BLOCKS;  // per block and part: one operand, 16 bytes a lane
    // block o of pair P, step kb >= P
    static constexpr int block(int P, int o, int kb) { return 2 * P * NK - P * (P - 1) + o * (NK - P) + kb - P; }
    // the matrix as operands, from its transpose, by THREADS threads, all loads at once; a barrier is the caller's
    template <int THREADS> static __device__ __forceinline__ void fill(char *to, const float *__restrict__ LinvT, int thread) {
        constexpr int N = (BLOCKS * 64 + THREADS - 1) / THREADS;
        float4 u[N], v[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int e = n * THREADS + thread, b = e >> 6, m = e & 15, q = e >> 4 & 3;
            if (e >= BLOCKS * 64) continue;
            int P = 0, first = 0;  // the pair and its first block
#pragma unroll
            for (int p = 1; p < NK; ++p)
                if (b >= block(p, 0, p)) {
                    P = p;
                    first = block(p, 0, p);
                }
            const int o = b - first >= NK - P, kb = P + b - first - o * (NK - P);
            const float *src = LinvT + (32 * P + 8 * (m >> 2) + 4 * o + (m & 3)) * D + 32 * kb + 8 * q;
            u[n] = *(const float4 *)src;
            v[n] = *(const float4 *)(src + 4);
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int e = n * THREADS + thread;
            if (e >= BLOCKS * 64) continue;
            bf16x8 part[PARTS];
            cut(u[n], v[n], part);
#pragma unroll
            for (int t = 0; t < PARTS; ++t) *(bf16x8 *)(to + (PARTS * (e >> 6) + t) * 1024 + (e & 63) * 16) = part[t];
        }
    }
    static __device__ __forceinline__ void cut(const float4 &u, const float4 &v, bf16x8 (&part)[PARTS]) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
        for (int t = 0; t < PARTS; ++t) {
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[e] = BF ? pack_nearest(x[2 * e], x[2 * e + 1]) : pack_upper(x[2 * e], x[2 * e + 1]);
                if (t + 1 < PARTS) {
                    x[2 * e] -= __uint_as_float(w[e] << 16);
                    x[2 * e + 1] -= __uint_as_float(w[e] & 0xffff0000u);
                }
            }
            part[t] = __builtin_bit_cast(bf16x8, w);
        }
    }
};

// The operands of pair P: block o, step kb and part t, from LDS or device memory.
template <int D, bool BF, int P> struct XOperands {
    using M = XMatrix<D, BF>;
    bf16x8 m[M::NK - P][2][M::PARTS];
    __device__ __forceinline__ void load(const char *mat, int lane) {
#pragma unroll
        for (int kb = P; kb < M::NK; ++kb)
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int t = 0; t < M::PARTS; ++t)
                    m[kb - P][o][t] = *(const bf16x8 *)(mat + lane * 16 + (M::PARTS * M::block(P, o, kb) + t) * 1024);
    }
};
// acc = columns 32 P + 8 q .. (four in [0], four in [1]) of the rows of NT tiles: xp[n][t][kb] is part t of the columns 32 kb + 8 q ..
// of row lane & 15 of tile n; step(kb) is called before the products of step kb and gives its operands [o][t].
template <int D, bool BF, int P, int NT, class Step>
__device__ __forceinline__ void x_pair(const bf16x8 (&xp)[NT][BF ? 2 : 3][D / 32], floatx4 (&acc)[NT][2], Step &&step) {
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n][0] = acc[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    static_for<P, D / 32>([&](auto kk) {
        constexpr int kb = decltype(kk)::value;
        const auto &m = step(kk);
        floatx4 s[NT][2];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int o = 0; o < 2; ++o) s[n][o] = BF ? acc[n][o] : floatx4{0.f, 0.f, 0.f, 0.f};
        static_for<0, BF ? 3 : 6>([&](auto xx) {  // small terms first; the chains of the tiles and blocks side by side
            constexpr int x = decltype(xx)::value + (BF ? 3 : 0);
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
            for (int o = 0; o < 2; ++o) acc[n][o] = BF ? s[n][o] : acc[n][o] + s[n][o];
    });
}

// NT tiles of sixteen rows, the matrix in LDS: store(n, P, x) gets the columns 32 P + 8 q .. of row lane & 15 of tile n.
template <int D, bool BF, int NT, class Store>
__device__ __forceinline__ void x_rows(const char *mat, const bf16x8 (&xp)[NT][BF ? 2 : 3][D / 32], Store &&store) {
    using M = XMatrix<D, BF>;
    const char *at = mat + (threadIdx.x & 63) * 16;
    static_for<0, M::NK>([&](auto pp) {
        constexpr int P = decltype(pp)::value;
        floatx4 acc[NT][2];
        bf16x8 m[2][M::PARTS];
        x_pair<D, BF, P, NT>(xp, acc, [&](auto kk) -> const auto & {
            constexpr int kb = decltype(kk)::value;
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int t = 0; t < M::PARTS; ++t) m[o][t] = *(const bf16x8 *)(at + (M::PARTS * M::block(P, o, kb) + t) * 1024);
            return m;
        });
#pragma unroll
        for (int n = 0; n < NT; ++n) store(n, P, acc[n]);
        __builtin_amdgcn_sched_barrier(0);  // keep the next pair's operand reads from piling up
    });
}

// The same for one tile with the matrix in device memory: the operands of the next pair are on their way while one pair's products
// are formed (left to itself the compiler waits for most of them one by one).  cut(xp) is called once the first pair's are.
template <int D, bool BF, class Cut, class Store>
__device__ __forceinline__ void x_rows_from_memory(const char *mat, int lane, Cut &&cut, Store &&store) {
    constexpr int NK = D / 32;
    bf16x8 xp[1][BF ? 2 : 3][NK];
    auto pair = [&](auto &self, const auto &now, auto pp) {
        constexpr int P = decltype(pp)::value;
        XOperands<D, BF, P + 1 < NK ? P + 1 : P> next;
        if constexpr (P + 1 < NK) next.load(mat, lane);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 acc[1][2];
        x_pair<D, BF, P, 1>(xp, acc, [&](auto kk) -> const auto & { return now.m[decltype(kk)::value - P]; });
        store(P, acc[0]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (P + 1 < NK) self(self, next, std::integral_constant<int, P + 1>{});
    };
    XOperands<D, BF, 0> first;
    first.load(mat, lane);
    __builtin_amdgcn_sched_barrier(0);
    cut(xp[0]);
    pair(pair, first, std::integral_constant<int, 0>{});
}

// the eight columns of a row that a lane holds, rounded to bf16 where the table is
template <bool BF> __device__ __forceinline__ void store_x8(typename std::conditional<BF, uint16_t, float>::type *dst, const floatx4 (&v)[2]) {
    if constexpr (BF) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        *(u32x4 *)dst = u32x4{pack_nearest(v[0][0], v[0][1]), pack_nearest(v[0][2], v[0][3]), pack_nearest(v[1][0], v[1][1]),
                              pack_nearest(v[1][2], v[1][3])};
    } else {
        *(floatx4 *)dst = v[0];
        *(floatx4 *)(dst + 4) = v[1];
    }
}

}  // namespace als
