// Dual row update for rows with 16 < k <= 32 stored entries.  The algebra is in the header comment of
// dual_prepare.hip.
#pragma once

#include "dual_walk.h"

namespace als {

// Four rows per wavefront, one per group of 16 lanes, each with a 32 x 32 system S = I + Z_I Z_I^T in 16 x 16 tiles
//     S = [ A  B^T ]      A: entries 0..15,  C: entries 16..31
//         [ B   C  ]
//   1. per row: gather its two tiles of entries into registers, form A, B, C on the matrix cores.  C stays in the
//      accumulator layout; A and B go to LDS and come back with lane i of a group holding rows i of A and of B;
//   2. sixteen steps of elimination on [A; B] in registers.  Every row of A but the pivot's is updated, the rows above
//      it too (Gauss-Jordan: those lanes would be idle otherwise), so A ends up diagonal and no triangular system is left
//      for a back-substitution; the right-hand side rides along.  Rows are scaled by the root of the pivot, L = B U^-1 P^1/2,
//      so that one operand serves both sides of step 3;
//   3. C -= L L^T on the fp32 matrix instruction, in place; C to one row per lane through LDS; sixteen steps of the same
//      elimination give t of the entries 16..31;
//   4. t of the entries 0..15: B^T t (columns of B from LDS, t as a DPP operand), the row operations of step 2 once more
//      on that vector (their multipliers were left where the eliminated columns were), and the pivots;
//   5. r = Z_I^T t, four (bf16: eight) columns per lane, from the registers of step 1, or (fp32, d = 128, whose tiles do not fit
//      the registers, and fp32 in the launch that small calls share) gathering the entries a second time; bf16 tables in the launch of
//      their own: X = R L^-1 of four steps' rows at a time (Parked, dual_walk.h).
// Every row goes through LDS into the operand layout (PieceGather), and the walk over the list loads the next step's ids ahead
// (dual_walk.h).
// What bounds it: HBM and the instructions of two wavefronts per SIMD, one every five clocks each, where the tiles stay in
// registers; with a second gather (fp32, d = 128) the latency of about twelve rounds of loads at three wavefronts per SIMD: on 10M
// pages 3.2 TB/s are counted.
// Per half, an elimination of all 32 columns in one block with a triangular back-substitution (616 multiply-adds with a DPP
// operand, 392 here) / this one with loads straight into the operand layout, 64 places per instruction / as it is:
//   50M power-law rows, bf16, d = 128  44.6 / 41.4 / 36.5 ms      10M pages, fp32, d = 128  7.65 / 7.15 / 6.35 ms
//   1M x 1M, fp32, d = 64 (second gather before)  705 / 671 / 525 us      300k rows, bf16, d = 128  129 / 115 / 107 us

// LDS of one wavefront: P holds four 16 x 16 tiles (A, then L, then C, then t), U the stage of two tiles of entries and later
// four tiles again (B); a block of zeros for slots beyond a row's k, the ids of the second gather.
// KEEP: rows of up to 256 bytes stay in registers.
template <int D, bool ZB, bool KEEP> struct MultiCfg {
    static constexpr int RB = D * ZT<ZB>::ES, CB = RB > 256 ? 256 : (KEEP || RB < 128 ? RB : 128), NCH = RB / CB;
    using PG = PieceGather<CB>;
    static constexpr int K = 32, TILE = TILE_FLOATS;
    static constexpr int OFF_P = 0, OFF_Q = 4 * TILE, U = 2 * PG::STAGE_FLOATS > 4 * TILE ? 2 * PG::STAGE_FLOATS : 4 * TILE;
    static constexpr int OFF_ZERO = OFF_Q + U, OFF_ID = OFF_ZERO + PG::ZERO_FLOATS;
    // what is loaded at a time: the chunk h of both tiles of row p is unit p * NCH + h.  RES: all units are loaded at once (128
    // registers at most) and stay in registers until r = Z_I^T t is formed from them, so nothing is gathered twice.  Otherwise
    // (fp32 with d = 128, whose rows are longer, and fp32 in the launch that small calls share, see dual_few.hip) two units are under way.
    static constexpr bool RES = KEEP && RB <= 256;
    static constexpr int UNITS = 4 * NCH, DEPTH = RES ? UNITS : 2;
    static constexpr int LDS_FLOATS = OFF_ID + (RES ? 0 : 4 * K);
    static constexpr int IDR = 2 * PG::N <= PG::IDS ? 1 : 2;  // id registers per row
    // where t and the id of entry e stand; with rows of up to 256 bytes the entries that a lane adds up stand side by side, in the
    // order in which RES has them, so that both forms have the same bits
    static constexpr bool SIDE = RB <= 256;
    static constexpr int PER_LANE = 2 * RowGather<D, ZB>::N;
    static __device__ __forceinline__ constexpr int slot(int e) { return SIDE ? e % RowGather<D, ZB>::EPI * PER_LANE + e / RowGather<D, ZB>::EPI : e; }
};

// (the members are what walk_steps and single_step want, see dual_walk.h)
template <int D, bool ZB, bool KEEP = true> struct MultiStep {
    using C = MultiCfg<D, ZB, KEEP>;
    using PG = typename C::PG;
    static constexpr int NIDS = 4 * C::IDR, N = PG::N, EPI = PG::EPI;
    static constexpr int LDS_FLOATS = C::LDS_FLOATS, FREE = C::OFF_Q;

    static __device__ __forceinline__ void init(float *lds, int lane) {
        if (lane < PG::ZERO_FLOATS) lds[C::OFF_ZERO + lane] = 0.f;
        static_assert(PG::ZERO_FLOATS <= 64, "one store a lane");
        wave_sync();
    }
    static __device__ __forceinline__ int id_entry(int lane, int r) { return C::IDR == 1 ? PG::id_entry(lane, 2 * N) : 16 * r + PG::id_entry(lane); }
    static __device__ __forceinline__ void ids(const int32_t *__restrict__ indices, const RowsDesc &d, int lane, int32_t (&idv)[NIDS]) {
#pragma unroll
        for (int n = 0; n < NIDS; ++n) {
            const int p = n / C::IDR, e = id_entry(lane, n % C::IDR);
            idv[n] = indices[d.b[p] + (e < d.k[p] ? e : 0)];  // clamped: a slot beyond k holds the row's first entry
        }
    }

    template <class Loaded, class Between, class Last, class Out>
    static __device__ __forceinline__ void solve(const float *__restrict__ values, const void *__restrict__ Z,
                                                 int32_t *__restrict__ err_flag, float *lds, const RowsDesc &d,
                                                 const int32_t (&idv)[NIDS], Loaded &&loaded, Between &&between, Last &&last, const Out &out) {
        constexpr int K = C::K;
        const int (&k)[4] = d.k;
        int kmax = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) kmax = k[p] > kmax ? k[p] : kmax;

        // ---- 1. gather and the tiles of S
        floatx4 z[C::DEPTH][2][N];  // (a float4 would be copied by way of scratch memory)
        const char *zlane = (const char *)Z + 16 * (opaque_tid() % PG::LPR);
        auto load = [&](auto uu) {
            constexpr int unit = decltype(uu)::value, p = unit / C::NCH, h = unit % C::NCH;
            static_for<0, 2>([&](auto tt) {
                static_for<0, N>([&](auto ss) {
                    constexpr int t = decltype(tt)::value, s = decltype(ss)::value;
                    // instructions that only meet slots beyond the row's k are left out (the first tile is full: k > 16)
                    if (t == 0 || 16 + s * EPI < k[p]) {
                        int32_t id;
                        if constexpr (C::IDR == 1) id = PG::template bcast_id<t * N + s>(idv[p]);
                        else id = PG::template bcast_id<s>(idv[2 * p + t]);
                        z[unit % C::DEPTH][t][s] = *(const floatx4 *)(zlane + (int64_t)id * C::RB + h * C::CB);
                    }
                });
            });
        };
        static_for<0, C::DEPTH>(load);
        loaded();
        const int lane = opaque_tid();  // after the loads: what derives from it is not kept across them
        const int a = lane & 15, q = lane >> 4;  // MFMA view: entry a of a tile, column group q
        const int g = lane >> 4, i = lane & 15;  // solver view: system g, lane i of its group
        // labels of the entries i and 16 + i of this lane's system
        float y0 = 0.f, y1 = 0.f;
        {
            int myk = 0;
            int64_t myb = 0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                myk = g == p ? k[p] : myk;
                myb = g == p ? d.b[p] : myb;
            }
            y0 = i < myk ? 1.f : 0.f;
            y1 = 16 + i < myk ? 1.f : 0.f;
            if (values) {
                int at = i;
                asm volatile("" : "+v"(at));  // no zero-extended copy of i across the step
                if (i < myk) y0 = values[myb + at];
                if (16 + i < myk) y1 = values[myb + at + 16];
            }
        }
        if constexpr (!C::RES) {
            int32_t *idl = (int32_t *)(lds + C::OFF_ID);
#pragma unroll
            for (int n = 0; n < NIDS; ++n) idl[n / C::IDR * K + C::slot(id_entry(lane, n % C::IDR))] = idv[n];
        }
        float *mfma_at = lds + tile_block(a, q);     // MFMA view: row a, columns 4 q .. of the first system's tile
        char *stage = (char *)(lds + C::OFF_Q);
        floatx4 cb[4], cc[4];
        static_for<0, 4>([&](auto pp) {
            constexpr int p = decltype(pp)::value;
            const floatx4 zero4 = floatx4{0.f, 0.f, 0.f, 0.f};
            floatx4 ca = zero4;
            cb[p] = zero4;
            cc[p] = zero4;
            static_for<0, C::NCH>([&](auto hh) {
                constexpr int unit = p * C::NCH + decltype(hh)::value;
                // what derives from the lane is formed again for each unit rather than kept
                const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;
                const int put = PG::put_base(lane), get = PG::get_base(a, q);
                static_for<0, 2>([&](auto tt) {
                    static_for<0, N>([&](auto ss) {
                        constexpr int t = decltype(tt)::value, s = decltype(ss)::value;
                        if (t == 0 || 16 + s * EPI < k[p])
                            *(floatx4 *)(stage + t * 16 * C::CB + PG::template put_at<s>(put)) = z[unit % C::DEPTH][t][s];
                    });
                });
                wave_sync();
                if constexpr (unit + C::DEPTH < C::UNITS) load(std::integral_constant<int, unit + C::DEPTH>{});
                // slots of the second tile beyond the row's k read zeros
                const bool have = 16 + a < k[p];
                const char *const zero = (const char *)(lds + C::OFF_ZERO);
                const char *at0[2] = {stage + get, stage + (get ^ 64)};
                const char *at1[2] = {have ? stage + 16 * C::CB + get : zero, have ? stage + 16 * C::CB + (get ^ 64) : zero};
                __builtin_amdgcn_s_setprio(1);  // matrix-core work first: other wavefronts fill in with vector work
                if constexpr (ZB) {
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        const bf16x8 o0 = *(const bf16x8 *)(at0[j & 1] + 128 * (j >> 1)), o1 = *(const bf16x8 *)(at1[j & 1] + 128 * (j >> 1));
                        ca = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o0, o0, ca, 0, 0, 0);
                        cb[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o0, o1, cb[p], 0, 0, 0);
                        cc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o1, o1, cc[p], 0, 0, 0);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < N; j += 2) {
                        const SplitOperand o0 = split_operand(*(const float4 *)(at0[0] + 64 * j), *(const float4 *)(at0[1] + 64 * j));
                        const SplitOperand o1 = split_operand(*(const float4 *)(at1[0] + 64 * j), *(const float4 *)(at1[1] + 64 * j));
                        ca = split_mfma(o0, o0, ca);
                        cb[p] = split_mfma(o0, o1, cb[p]);
                        cc[p] = split_mfma(o1, o1, cc[p]);
                    }
                }
                __builtin_amdgcn_s_setprio(0);
                wave_sync();  // the next unit reuses the stage
            });
            // ca[v] = A[a][4 q + v], cb[p][v] = B[a][4 q + v], cc[p][v] = C[a][4 q + v] (A and C are symmetric)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float one = 4 * q + v == a ? 1.f : 0.f;
                ca[v] += one;
                cc[p][v] += one;
            }
            *(floatx4 *)(mfma_at + C::OFF_P + p * C::TILE) = ca;
        });
        between();
#pragma unroll
        for (int p = 0; p < 4; ++p) *(floatx4 *)(mfma_at + C::OFF_Q + p * C::TILE) = cb[p];
        wave_sync();

        // ---- 2. elimination of the columns of A
        float *row_at = lds + g * C::TILE + 16 * i;  // solver view: row i of system g
        const int swz = (i >> 1 & 3) << 2;           // block b of that row lies at row_at + (4 b ^ swz)
        float s0[16], s1[16], ri0 = 1.f, ri1 = 1.f;
        bool bad = false;
        load_tile_row(row_at + C::OFF_P, i, s0);
        load_tile_row(row_at + C::OFF_Q, i, s1);
        dpp_settle(s0[0]);
        static_for<0, 16>([&](auto ci) { eliminate_column<decltype(ci)::value>(s0, y0, ri0, i, bad, RowBelow{s1, y1}); });

        // ---- 3. C - L L^T and its elimination
        wave_sync();  // every lane has read its rows of A
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4)
            *(float4 *)(row_at + C::OFF_P + (4 * c4 ^ swz)) = make_float4(s1[4 * c4], s1[4 * c4 + 1], s1[4 * c4 + 2], s1[4 * c4 + 3]);
        wave_sync();
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            // lane (a, q) supplies L[a][4 q + e] to instruction e on both sides: the contraction runs over all 16 columns
            const floatx4 o = *(const floatx4 *)(mfma_at + C::OFF_P + p * C::TILE);
#pragma unroll
            for (int e = 0; e < 4; ++e) cc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(-o[e], o[e], cc[p], 0, 0, 0);
        }
        wave_sync();
#pragma unroll
        for (int p = 0; p < 4; ++p) *(floatx4 *)(mfma_at + C::OFF_P + p * C::TILE) = cc[p];
        float bt[16];  // column i of B
#pragma unroll
        for (int m = 0; m < 16; ++m)
            bt[m] = lds[C::OFF_Q + g * C::TILE + 16 * m + (((i >> 2) ^ (m >> 1) & 3) << 2) + (i & 3)];
        wave_sync();
        load_tile_row(row_at + C::OFF_P, i, s1);
        dpp_settle(s1[0]);
        static_for<0, 16>([&](auto ci) {
            constexpr int c = decltype(ci)::value;
            if (16 + c < kmax) eliminate_column<c>(s1, y1, ri1, i, bad);  // beyond every row's k: identity rows
        });
        // a row past the end of the list stands for the step's first entry sixteen times over (its first tile is not masked): its
        // pivots mean nothing
        const int rel_lo = g & 1 ? d.row.rel[1] : d.row.rel[0], rel_hi = g & 1 ? d.row.rel[3] : d.row.rel[2];
        if (bad && (g & 2 ? rel_hi : rel_lo) >= 0) atomicOr(err_flag, 1);

        // ---- 4. t of both halves
        float t1 = y1 * ri1 * ri1;
        float za = 0.f, zb = 0.f;
        dpp_settle(t1);
        static_for<0, 8>([&](auto mm) {
            constexpr int m = decltype(mm)::value;
            fmac_bcast16<2 * m>(za, t1, bt[2 * m]);
            fmac_bcast16<2 * m + 1>(zb, t1, bt[2 * m + 1]);
        });
        za += zb;
        static_for<0, 16>([&](auto ci) {
            constexpr int c = decltype(ci)::value;
            dpp_settle(za);
            fmac_bcast16_neg<c>(za, za, s0[c]);
        });
        const float t0 = (y0 - za) * ri0 * ri0;
        wave_sync();  // every lane has read its row of C
        if constexpr (C::RES) {
            // ---- 5. r = Z_I^T t from the registers of step 1, four (bf16: eight) columns per lane
            float *tb = lds + C::OFF_P;  // t of the entries of one lane side by side
            tb[g * K + C::slot(i)] = t0;
            tb[g * K + C::slot(i) + C::slot(16)] = t1;
            wave_sync();
            constexpr int NV = ZB ? 2 : 1;
            floatx4 rv[4][NV];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float *tp = tb + p * K + lane / PG::LPR * 2 * N;
                float t[2 * N];
                if constexpr (N >= 2) {
#pragma unroll
                    for (int h = 0; h < N / 2; ++h) {
                        const float4 v = ((const float4 *)tp)[h];
                        t[4 * h] = v.x; t[4 * h + 1] = v.y; t[4 * h + 2] = v.z; t[4 * h + 3] = v.w;
                    }
                } else {
                    t[0] = tp[0];
                    t[1] = tp[1];
                }
#pragma unroll
                for (int n = 0; n < NV; ++n) rv[p][n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int x = 0; x < 2 * N; ++x) {
                    if (x >= N && 16 + (x - N) * EPI >= k[p]) continue;  // uniform
                    const floatx4 w = z[p % C::DEPTH][x / N][x % N];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        if constexpr (ZB) {
                            rv[p][c / 2][2 * (c & 1)] += t[x] * __uint_as_float(__float_as_uint(w[c]) << 16);
                            rv[p][c / 2][2 * (c & 1) + 1] += t[x] * __uint_as_float(__float_as_uint(w[c]) & 0xffff0000u);
                        } else {
                            rv[p][0][c] += t[x] * w[c];
                        }
                    }
                }
            }
            last();
            out.template store<PG::LPR>(rv, lane);
            return;
        }
        if constexpr (!C::RES) {
        const int32_t *ids = (const int32_t *)(lds + C::OFF_ID);
        float *tbuf = lds + C::OFF_P;
        tbuf[g * K + C::slot(i)] = t0;
        tbuf[g * K + C::slot(i) + C::slot(16)] = t1;
        wave_sync();

        // ---- 5. r = Z_I^T t (second gather of the row's entries): 16 bytes of an entry per lane, so that one instruction takes
        // GatherCols<D>::EPI entries; the four rows advance together, EPL entries per lane and round.  Per round: first the
        // ids and t of all rows from LDS, then the loads, then the products - no wait and no lane-dependent branch between
        // two loads.
        {
            using GC = GatherCols<D>;
            constexpr int EPL = 4, EPR = EPL * GC::EPI;
            // round e0 / EPR takes the entries e0 .. e0 + EPR - 1
            const int mine = (C::SIDE ? C::PER_LANE : EPL) * (lane / GC::LPR);
            const float *col = (const float *)Z + 4 * (lane % GC::LPR);
            floatx4 rv[4][1];
#pragma unroll
            for (int p = 0; p < 4; ++p) rv[p][0] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int e0 = 0; e0 < kmax; e0 += EPR) {  // padded entries have t = 0 and the id of the row's first entry
                typedef int intv __attribute__((ext_vector_type(EPL)));
                typedef float floatv __attribute__((ext_vector_type(EPL)));
                intv id[4];
                floatv te[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int at = p * K + mine + (C::SIDE ? e0 / GC::EPI : e0);
                    id[p] = *(const intv *)(ids + at);
                    te[p] = *(const floatv *)(tbuf + at);
                }
                floatx4 zz[4][EPL];
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (e0 < k[p]) {  // uniform
#pragma unroll
                        for (int x = 0; x < EPL; ++x) zz[p][x] = *(const floatx4 *)(col + (int64_t)id[p][x] * D);
                    }
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (e0 < k[p]) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int x = 0; x < EPL; ++x) rv[p][0][c] += te[p][x] * zz[p][x][c];
                    }
            }
            last();
            out.template store<GC::LPR>(rv, lane);
        }
        }
    }
};

template <int D, bool ZB, bool KEEP>
__device__ __forceinline__ void dual_multi_step(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                const float *__restrict__ values, const void *__restrict__ Z,
                                                float *__restrict__ R, int64_t ldr, int64_t r0,
                                                const int32_t *__restrict__ list, int count,
                                                int32_t *__restrict__ err_flag, int blk, float *lds) {
    single_step<MultiStep<D, ZB, KEEP>>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
}

}  // namespace als
