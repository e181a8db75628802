// The shared factor of the dual row update (see the header comment of dual_prepare.hip).
#pragma once

#include "dual_common.h"

namespace als {

// B = alpha*G + lambda*I -> L^{-1} (B = L L^T) in fp64, one workgroup.  Outputs Linv (row-major, zeros above the
// diagonal) and its transpose LinvT, both fp32 [D*D].
//
// What bounds it is the chain of D dependent pivots, so everything else is taken off that chain: the matrix is
// worked in blocks of 16 columns, B = M P M^T with M unit lower triangular (no square root and no division
// between two pivots: a reciprocal by two Newton steps).  Per block column p:
//   wavefront 0 eliminates the 16 x 16 diagonal block in registers, in place: a column that is done makes room for the
//     same column of the inverse of the block's M.  Lane (i, q) owns the entries (i, 4 s + q), so that a step takes four
//     multiply-adds; the pivot column crosses the rows of 16 lanes with lane swaps, the pivot row comes by row broadcasts.
//   the blocks below become W = A M_pp^{-T} (= M P), one per wavefront
//   wavefront 0 updates the next diagonal block and goes on with its elimination, while the others work off the rest of
//     the trailing blocks, A_ij -= W_i P^{-1} W_j^T, on the fp64 matrix cores and row p of the inverse of M
//     (N_pj = -N_pp sum_k M_pk N_kj; kept in the upper blocks of the same LDS array).
// L^{-1} = P^{-1/2} M^{-1}.
// D = 128: 600 us as an element-wise Cholesky with a barrier per column, 48 us with these stages one after the other and sixteen
// multiply-adds per step, 31 us in this form (d = 64: 158, 21 and 15 us; d = 16: 15, 4.3 and 3.7 us).
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int FACTOR_THREADS = 512;

template <int D> struct FactorCfg {
    static constexpr int NB = D / 16, LD = D + 1;
    static constexpr int OFF_N = D * LD;               // inverses of the diagonal blocks of M, [NB][16][17]
    static constexpr int OFF_RP = OFF_N + NB * 16 * 17;  // reciprocal pivots [D], then their roots [D]
    static constexpr size_t LDS_BYTES = (size_t)(OFF_RP + 2 * D) * sizeof(double);
};

__device__ __forceinline__ double from_words(uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t low_word(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t high_word(double v) { return (uint32_t)(__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double lane_value_f64(double v, int src_lane) {
    return from_words(__builtin_amdgcn_readlane((int)low_word(v), src_lane), __builtin_amdgcn_readlane((int)high_word(v), src_lane));
}
// value of lane C of this lane's row of 16 lanes
template <int C> __device__ __forceinline__ double bcast16_f64(double v) {
    return from_words(__builtin_amdgcn_update_dpp(0, (int)low_word(v), 0x150 + C, 0xf, 0xf, true),
                      __builtin_amdgcn_update_dpp(0, (int)high_word(v), 0x150 + C, 0xf, 0xf, true));
}
template <int Q> __device__ __forceinline__ double from_lane_row_f64(double v) {
    return from_words(from_lane_row<Q>(low_word(v)), from_lane_row<Q>(high_word(v)));
}

// One wavefront: the 16 x 16 block at `blk` (rows LD apart, lower triangle) -> nd[16][17] = inverse of its unit lower M,
// rp[16] = reciprocal pivots.
template <int LD>
__device__ __forceinline__ void factor_block(const double *blk, double *nd, double *rp_out, int32_t *__restrict__ err_flag) {
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    double x[4], mine = 1.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int j = 4 * s + q;
        x[s] = blk[(j <= i ? i : j) * LD + (j <= i ? j : i)];
    }
    bool bad = false;
    static_for<0, 16>([&](auto cc) {
        constexpr int c = decltype(cc)::value, sc = c / 4, qc = c % 4;
        const double pivot = lane_value_f64(x[sc], 16 * qc + c);
        bad |= !(pivot > 0.0);
        double rp = __builtin_amdgcn_rcp(pivot);
        rp = rp * (2.0 - pivot * rp);
        rp = rp * (2.0 - pivot * rp);
        mine = i == c ? rp : mine;
        const double col = from_lane_row_f64<qc>(x[sc]);
        const double f = i > c ? col * rp : 0.0;
        const double done = i == c ? 1.0 : -f;  // this row's entry of the inverse in column c
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double next = x[s] - f * bcast16_f64<c>(x[s]);
            x[s] = s == sc && q == qc ? done : next;
        }
    });
    if (bad && lane == 0) atomicOr(err_flag, 1);
#pragma unroll
    for (int s = 0; s < 4; ++s) nd[i * 17 + 4 * s + q] = x[s];
    if (q == 0) rp_out[i] = mine;
}

// By FACTOR_THREADS threads, with FactorCfg<D>::LDS_BYTES of LDS.
template <int D>
__device__ __forceinline__ void factor(const float *__restrict__ G, float alpha, float lambda, float *__restrict__ Linv,
                                       float *__restrict__ LinvT, int32_t *__restrict__ err_flag, double *fa) {
    using C = FactorCfg<D>;
    constexpr int NB = C::NB, LD = C::LD, T = FACTOR_THREADS, NW = T / 64, PER = (D * D + T - 1) / T;
    static_assert(NB <= NW, "one wavefront per block of a column, and one more while the last row of N is formed");
    double *a = fa, *nd = fa + C::OFF_N, *rpb = fa + C::OFF_RP, *root = rpb + D;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int i16 = lane & 15, q = lane >> 4;
    {
        float g[PER];  // all in flight together
#pragma unroll
        for (int n = 0; n < PER; ++n)
            if (n * T + t < D * D) g[n] = G[n * T + t];
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            const int e = n * T + t, r = e / D, c = e % D;
            if (e < D * D) a[r * LD + c] = (double)alpha * (double)g[n] + (r == c ? (double)lambda : 0.0);
        }
    }
    __syncthreads();
    // v_mfma_f64_16x16x4: lane (i16, q) supplies A[i16][q] and B[q][i16] and holds C[q + 4 v][i16]; the depth step s
    // contracts the block's columns 4 s + q
    auto trailing = [&](int p, int e) {  // A_ij -= W_i P^{-1} W_j^T for block e of the trailing lower triangle
        int bi = 0, rest = e;
        while (rest > bi) rest -= ++bi;
        const int i = p + 1 + bi, j = p + 1 + rest;
        doublex4 acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = a[(16 * i + q + 4 * v) * LD + 16 * j + i16];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = 16 * p + 4 * s + q;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[(16 * i + i16) * LD + k] * rpb[k], a[(16 * j + i16) * LD + k], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) a[(16 * i + q + 4 * v) * LD + 16 * j + i16] = acc[v];
    };
    auto inverse = [&](int i, int j) {  // N_ij, j < i, from rows j .. i - 1 of N; kept in the free upper block (j, i)
        doublex4 s4 = {0.0, 0.0, 0.0, 0.0};
        for (int k = j; k < i; ++k) {
            const double *nk = k == j ? nd + j * 16 * 17 : a + 16 * j * LD + 16 * k;
            const int nld = k == j ? 17 : LD;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int c = 16 * k + 4 * s + q;
                s4 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(16 * i + i16) * LD + c] * rpb[c], nk[(4 * s + q) * nld + i16], s4, 0, 0, 0);
            }
        }
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s)  // the sum's accumulator layout is the B operand's
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-nd[(i * 16 + i16) * 17 + 4 * s + q], s4[s], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) a[(16 * j + q + 4 * v) * LD + 16 * i + i16] = acc[v];
    };
    if (wave == 0) factor_block<LD>(a, nd, rpb, err_flag);
    __syncthreads();
    for (int p = 0; p + 1 < NB; ++p) {
        // W_i = A_ip N_pp^T, in place
        const int w = p + 1 + wave;
        if (w < NB) {
            doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(16 * w + i16) * LD + 16 * p + 4 * s + q],
                                                           nd[(p * 16 + i16) * 17 + 4 * s + q], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) a[(16 * w + q + 4 * v) * LD + 16 * p + i16] = acc[v];
        }
        __syncthreads();
        if (wave == 0) {
            const int n = p + 1;
            trailing(p, 0);
            wave_sync();
            factor_block<LD>(a + 16 * n * (LD + 1), nd + n * 16 * 17, rpb + 16 * n, err_flag);
        } else {
            const int TB = NB - p - 1, tiles = TB * (TB + 1) / 2 - 1;
            for (int u = wave - 1; u < p + tiles; u += NW - 1) {
                if (u < p) inverse(p, u);
                else trailing(p, u - p + 1);
            }
        }
        __syncthreads();
    }
    if (wave < NB - 1) inverse(NB - 1, wave);
    else if (wave == NW - 1)
        for (int r = lane; r < D; r += 64) root[r] = sqrt(rpb[r]);  // a pivot that was not positive leaves NaN here; the flag is set
    __syncthreads();
    auto entry = [&](int r, int c) {  // L^{-1}[r][c]
        const int br = r >> 4, bc = c >> 4;
        const double *n = br == bc ? nd + r * 17 + (c & 15) : a + (16 * bc + (r & 15)) * LD + 16 * br + (c & 15);
        return c > r ? 0.f : (float)(*n * root[r]);
    };
#pragma unroll 8
    for (int n = 0; n < PER; ++n) {
        const int e = n * T + t, r = e / D, c = e % D;
        if (e < D * D) {
            Linv[e] = entry(r, c);
            LinvT[e] = entry(c, r);
        }
    }
}

}  // namespace als
