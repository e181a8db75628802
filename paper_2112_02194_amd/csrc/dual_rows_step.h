// Dual row update for rows with 8 < k <= 16 stored entries: four rows per wavefront, one lane per row of
// the k x k system.  The algebra is in the header comment of dual_prepare.hip.
#pragma once

#include "dual_walk.h"

namespace als {

// One wavefront (= one workgroup) solves four rows taken from `list` (row ids relative to r0), all
// with at most 16 stored entries:
//   1. the entries of all four rows are loaded into registers, side-by-side lanes side-by-side pieces of an entry; tile by
//      tile they go through LDS into the operand layout (RowGather) and S = I + Z_I Z_I^T is formed on the matrix cores;
//   2. lane i of a row's group of 16 lanes owns row i of S: Gauss-Jordan elimination with DPP broadcasts inside the group, the
//      right-hand side riding along, so that nothing is left for a triangular solve;
//   3. r = Z_I^T t from the registers of step 1, four (bf16: eight) columns per lane, summed over the lanes that hold
//      other entries of the same columns.
// What bounds it: HBM where the columns are spread (50M rows, fp32).  On 10M pages of locality (d = 128, fp32) loads straight
// into the operand layout kept the data units busy 89% of the time, and 57% of a wavefront's life was spent waiting for four
// dependent loads.  Per half, before / with the gather through LDS and without the triangular solves / walking the list with
// loads ahead (dual_walk.h): 10M pages 3.40 / 2.99 / 2.64 ms, 50M rows fp32 11.0 / 11.1 / 10.5 ms, 1M x 1M (d = 64) 118 / 98 /
// 85 us, 300k bf16 rows (d = 128) 62 / 52 / 50 us.
template <int D, bool ZB> struct RowsCfg {
    using RG = RowGather<D, ZB>;
    static constexpr int RPW = 4;  // rows per wavefront (read as one ListQuad)
    static constexpr int OFF_ZERO = RG::STAGE_FLOATS, OFF_S = OFF_ZERO + RG::ZERO_FLOATS, OFF_T = OFF_S + 4 * TILE_FLOATS;
    static constexpr int LDS_FLOATS = OFF_T + 64;
};

// (the members are what walk_steps and single_step want, see dual_walk.h)
template <int D, bool ZB> struct RowsStep {
    static constexpr int NIDS = 4, LDS_FLOATS = RowsCfg<D, ZB>::LDS_FLOATS, FREE = 0;
    // Where S is formed in full fp32 precision (d = 16), the rounding of the elimination is what is left, and the Gauss-Jordan form
    // rounds a little more than triangular solves do.  Error against fp64, 8 < k <= 16, fp32, alpha = 0.05 / 1e-4 / 1e-5: triangular
    // 1.79e-7 / 3.80e-7 / 1.12e-6, Gauss-Jordan 1.76e-7 / 4.04e-7 / 1.15e-6, with one step of refinement 1.32e-7 / 3.25e-7 / 0.97e-6;
    // 300k such rows 145 -> 152 us (153 with the triangular solves).  With d >= 32 the cut operands of S (fp32) or the rounding of
    // the result (bf16) decide: all forms agree to 0.2 %.
    static constexpr bool REFINE = D == 16;
    // the zeros that slots beyond a row's k read
    static __device__ __forceinline__ void init(float *lds, int lane) {
        using C = RowsCfg<D, ZB>;
#pragma unroll
        for (int e = 0; e < C::RG::ZERO_FLOATS; e += 64)
            if (e + lane < C::RG::ZERO_FLOATS) lds[C::OFF_ZERO + e + lane] = 0.f;
        wave_sync();
    }
    // column ids in the order of RowGather
    static __device__ __forceinline__ void ids(const int32_t *__restrict__ indices, const RowsDesc &d, int lane, int32_t (&idv)[NIDS]) {
        const int e = RowGather<D, ZB>::id_entry(lane);
#pragma unroll
        for (int p = 0; p < 4; ++p) idv[p] = indices[d.b[p] + (e < d.k[p] ? e : 0)];  // clamped: rows of the class have k >= 1
    }
    template <class Loaded, class Between, class Last, class Out>
    static __device__ __forceinline__ void solve(const float *__restrict__ values, const void *__restrict__ Z,
                                                 int32_t *__restrict__ err_flag, float *lds, const RowsDesc &d,
                                                 const int32_t (&idv)[NIDS], Loaded &&loaded, Between &&between, Last &&last, const Out &out) {
        using C = RowsCfg<D, ZB>;
        using RG = RowGather<D, ZB>;
        constexpr int RPW = C::RPW, N = RG::N, EPI = RG::EPI;
        const int (&k)[4] = d.k;
        float *zero = lds + C::OFF_ZERO, *sm = lds + C::OFF_S, *tb = lds + C::OFF_T;
        int kmax = 0;
#pragma unroll
        for (int p = 0; p < RPW; ++p) kmax = k[p] > kmax ? k[p] : kmax;

        // ---- 1. gather and S tiles
        // All loads of the step are issued before the first one is waited for; instructions that only meet slots beyond the row's k
        // are left out (the class has k > 8), a slot beyond k inside an instruction loads the row's first entry (and meets t = 0).
        float4 z[RPW][N];
        const char *zlane = (const char *)Z + 16 * (opaque_tid() % RG::LPR);
#pragma unroll
        for (int p = 0; p < RPW; ++p) {
            static_for<0, N>([&](auto ss) {
                constexpr int s = decltype(ss)::value;
                if ((s + 1) * EPI <= 9 || s * EPI < k[p]) z[p][s] = *(const float4 *)(zlane + (int64_t)RG::template bcast_id<s>(idv[p]) * RG::RB);
            });
            if constexpr (N > 4) __builtin_amdgcn_sched_barrier(0);  // d = 128, fp32: every register counts
        }
        loaded();
        const int lane = opaque_tid();  // after the loads: what derives from it is not kept across them
        const int a = lane & 15, q = lane >> 4;  // MFMA view: entry a of a tile, column group q
        const int g = lane >> 4, i = lane & 15;  // solver view: system g, lane i of its group
        float y;  // label of entry i of this lane's system
        {
            int myk = 0;
            int64_t myb = 0;
#pragma unroll
            for (int p = 0; p < RPW; ++p) {
                myk = g == p ? k[p] : myk;
                myb = g == p ? d.b[p] : myb;
            }
            y = i < myk ? 1.f : 0.f;
            if (values) {
                int at = i;
                asm volatile("" : "+v"(at));  // no zero-extended copy of i across the step: a register too many at d = 128
                y = i < myk ? values[myb + at] : 0.f;
            }
        }
        char *stage = (char *)lds;
#pragma unroll
        for (int p = 0; p < RPW; ++p) {
            // what derives from the lane is formed again for each tile rather than kept: a dozen registers, which at d = 128 (fp32)
            // would cost a wavefront per SIMD
            const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;
            const int put = RG::put_base(lane), get = RG::get_base(a, q);
            static_for<0, N>([&](auto ss) {
                constexpr int s = decltype(ss)::value;
                if ((s + 1) * EPI <= 9 || s * EPI < k[p]) *(float4 *)(stage + RG::template put_at<s>(put)) = z[p][s];
            });
            wave_sync();
            // slots beyond the row's k read zeros
            const bool have = a < k[p];
            const char *even = have ? stage + get : (const char *)zero;
            const char *odd = have ? stage + (get ^ 64) : (const char *)zero;
            floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
            // two pieces at a time at d = 128: the registers of a tile in operand layout beside four tiles as loaded would cost a wavefront per SIMD
            constexpr int NO = N < 8 ? N : 2;
#pragma unroll
            for (int j0 = 0; j0 < N; j0 += NO) {
                float4 o[NO];
#pragma unroll
                for (int j = 0; j < NO; ++j) o[j] = *(const float4 *)((j & 1 ? odd : even) + 128 * ((j0 + j) >> 1));
                if constexpr (ZB) {  // bf16 rows are matrix-core operands as loaded
                    acc = mfma_pieces_bf16<NO>(o, o, acc);
                } else if constexpr (N >= 2) {  // split products on the bf16 matrix cores
#pragma unroll
                    for (int h = 0; h < NO / 2; ++h) {
                        const SplitOperand zs = split_operand(o[2 * h], o[2 * h + 1]);
                        acc = split_mfma(zs, zs, acc);
                    }
                } else {
                    const float c[4] = {o[0].x, o[0].y, o[0].z, o[0].w};
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c[v], c[v], acc, 0, 0, 0);
                }
                if constexpr (N > 4) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += 4 * q + v == a ? 1.f : 0.f;  // S[a][4 q + v] (S is symmetric)
            *(floatx4 *)(sm + p * TILE_FLOATS + tile_block(a, q)) = acc;
            wave_sync();  // the next tile reuses the stage
        }

        between();

        // ---- 2. elimination
        float s[16], ri = 1.f;
        bool bad = false;
        const float label = y;
        load_tile_row(sm + g * TILE_FLOATS + 16 * i, i, s);
        dpp_settle(s[0]);
        static_for<0, 16>([&](auto ci) {
            constexpr int c = decltype(ci)::value;
            if (c < kmax) eliminate_column<c>(s, y, ri, i, bad);  // beyond every row's k: identity rows
        });
        if (bad) atomicOr(err_flag, 1);
        float t = y * ri * ri;
        if constexpr (REFINE) {  // t += S^-1 (label - S t); the multipliers of the row operations were left in s
            float row[16], r0 = label, r1 = 0.f;
            load_tile_row(sm + g * TILE_FLOATS + 16 * i, i, row);
            dpp_settle(t);
            static_for<0, 8>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                fmac_bcast16_neg<2 * m>(r0, t, row[2 * m]);
                fmac_bcast16_neg<2 * m + 1>(r1, t, row[2 * m + 1]);
            });
            r0 += r1;
            static_for<0, 16>([&](auto ci) {
                constexpr int c = decltype(ci)::value;
                if (c < kmax) {
                    dpp_settle(r0);
                    fmac_bcast16_neg_self<c>(r0, s[c]);
                }
            });
            const float more = r0 * ri * ri;
            t += fabsf(more) < __builtin_inff() ? more : 0.f;  // not where the residual has left the range of numbers
        }
        tb[16 * g + i % EPI * N + i / EPI] = t;  // t of the entries of one lane side by side
        wave_sync();

        // ---- 3. r = Z_I^T t
        constexpr int NV = ZB ? 2 : 1;
        floatx4 rv[RPW][NV];
#pragma unroll
        for (int p = 0; p < RPW; ++p) {
            const float *tp = tb + 16 * p + lane / RG::LPR * N;
            float t[N];
            if constexpr (N >= 4) {
#pragma unroll
                for (int h = 0; h < N / 4; ++h) {
                    const float4 v = ((const float4 *)tp)[h];
                    t[4 * h] = v.x; t[4 * h + 1] = v.y; t[4 * h + 2] = v.z; t[4 * h + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int h = 0; h < N; ++h) t[h] = tp[h];
            }
            if (N > 4 && p == RPW - 1)  // d = 128, fp32: the last tile is still in the stage, its registers were free for the solver
                static_for<0, N>([&](auto ss) {
                    constexpr int s = decltype(ss)::value;
                    z[p][s] = *(const float4 *)(stage + RG::template put_at<s>(RG::put_base(lane)));
                });
#pragma unroll
            for (int n = 0; n < NV; ++n) rv[p][n] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (N > 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < N; ++x) {
                if ((x + 1) * EPI > 9 && x * EPI >= k[p]) continue;
                const float w[4] = {z[p][x].x, z[p][x].y, z[p][x].z, z[p][x].w};
                if constexpr (ZB) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        rv[p][c / 2][2 * (c & 1)] += t[x] * __uint_as_float(__float_as_uint(w[c]) << 16);
                        rv[p][c / 2][2 * (c & 1) + 1] += t[x] * __uint_as_float(__float_as_uint(w[c]) & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) rv[p][0][c] += t[x] * w[c];
                }
            }
        }
        last();
        out.template store<RG::LPR>(rv, lane);
    }
};

template <int D, bool ZB>
__device__ __forceinline__ void dual_rows_step(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                               const float *__restrict__ values, const void *__restrict__ Z,
                                               float *__restrict__ R, int64_t ldr, int64_t r0,
                                               const int32_t *__restrict__ list, int count,
                                               int32_t *__restrict__ err_flag, int blk, float *lds) {
    single_step<RowsStep<D, ZB>>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
}

}  // namespace als
