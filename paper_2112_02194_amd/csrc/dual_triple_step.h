// Dual row update for rows with 32 < k <= 48 stored entries.  The algebra is in the header comment of dual_prepare.hip.
#pragma once

#include "dual_walk.h"

namespace als {

// One step of the eliminations with the rows of a block column spread over the wavefront: the lanes below TOP (16 or 32) hold the rows of the
// pivots' block, 16 lanes each, the others rows below it.  The operations on a row are those of eliminate_column.
template <int c, int TOP>
__device__ __forceinline__ void eliminate_shared(float (&s)[16], float &y, float &rinv, int lane, bool &bad) {
    const float pivot = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s[c]), c));
    const float uc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), c));
    bad |= !(pivot > 0.f);
    float ri = __builtin_amdgcn_rsqf(pivot);
    ri = ri * (1.5f - 0.5f * pivot * ri * ri);  // one Newton step on the hardware estimate
    float l = (TOP == 16 ? from_lane_row<0>(s[c]) : from_lower_half(s[c])) * ri;
    const bool top = lane < TOP, pivots = (lane & 15) == c;
    const float mine = s[c] * ri, own = top && pivots ? 0.f : mine, w = uc * ri;
    rinv = pivots ? ri : rinv;
    y -= own * w;
    dpp_settle(l);  // just written, read through DPP below
    static_for<c + 1, 16>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        fmac_bcast16_neg<j>(s[j], l, own);
    });
    s[c] = top ? own * ri : mine;
    if constexpr (c + 1 < 16) dpp_settle(s[c + 1]);  // read across lanes by the next step
}

// Four rows per wavefront, one per group of 16 lanes, each with a 48 x 48 system S = I + Z_I Z_I^T in 16 x 16 tiles S_ij; the steps
// of 16 < k <= 32 (dual_multi_step.h) with a block more:
//   1. per row: the entries go through LDS into the operand layout (PieceGather) and the six tiles of the lower triangle are formed
//      on the matrix cores.  S_11, S_21 and S_22 stay in the accumulator layout, the tiles of the first block column go to LDS and come
//      back with lane i of a group holding row i of each;
//   2. sixteen Gauss-Jordan steps on the first block column in registers (S_00 becomes diagonal, the multipliers stay where
//      the eliminated columns were), the other tiles -= L_i L_j^T on the fp32 matrix instruction; the same for the second block
//      column, and sixteen steps on what is left of S_22;
//   3. t of the last block, and backwards t_p = S_pp^-1 (y_p - sum S_ip^T t_i): columns of S_ip from LDS, t as a DPP operand, the
//      row operations of S_pp once more;
//   4. r = Z_I^T t, gathering the entries a second time, 16 bytes a lane.
// R = 1: one row per wavefront, for the launch that small calls share, whose rows are too few for more, with the same operations on a row
// in the same order: the rows of a block column are spread over the groups of 16 lanes, the last 16 x 16 system stands in all of them.
// (With the same system in every group, the common launch of 15 000 rows of 40 entries took 67.4 us at d = 64, fp32, and 61.8 for bf16, now 61.6
// and 57.6, of 9000 rows 45.8 and 40.0, now 42.9 and 37.6; with a triangle in LDS 63.7, 56.3, 43.6 and 38.0.)
// What bounds it: the instructions of two wavefronts per SIMD (about 16 000 clocks a step of four rows at 64 columns, with 800 multiply-adds
// with a DPP operand at half rate) and what they wait for memory in between; R = 1: the chain of 48 steps.
// Against one row per wavefront and a triangle in LDS (tri_solve.h), per epoch: 10M pages, fp32, d = 128 5.15 -> 4.70 ms; 1M x 1M, fp32,
// d = 64 1089 -> 880 us; 50M power-law rows, bf16, d = 128 19.3 -> 16.6 ms.  The entries' second gather starting before the solve and
// running two rounds ahead is 6 to 10 % of that.
template <int D, bool ZB, int R> struct TripleCfg {
    static constexpr int RB = D * ZT<ZB>::ES, CB = RB < 256 / (R == 4 ? 1 : 2) ? RB : 256 / (R == 4 ? 1 : 2), NCH = RB / CB;
    using PG = PieceGather<CB>;
    static constexpr int AREA = R * TILE_FLOATS;  // a tile per row
    // T: S_00, then L_10, S_11, L_21, S_22 and t; then S_10, S_20 and (before that L_20) S_21, at first the stage of three tiles of entries
    static constexpr int OFF_T = 0, OFF_10 = AREA, OFF_20 = 2 * AREA, OFF_21 = 3 * AREA;
    static constexpr int U = 3 * AREA > 3 * PG::STAGE_FLOATS ? 3 * AREA : 3 * PG::STAGE_FLOATS;
    static constexpr int OFF_ZERO = OFF_10 + U, OFF_ID = OFF_ZERO + PG::ZERO_FLOATS;
    static constexpr int KS = 64;                 // places of a row's ids and t
    static_assert(R * KS <= AREA, "t takes the place of S_22");
    static constexpr int LDS_FLOATS = OFF_ID + R * KS;
    static constexpr int UNITS = R * NCH, DEPTH = R == 4 ? 2 : UNITS;  // a unit: one chunk of a row's three tiles
    static constexpr int IDR = (3 * PG::N + PG::IDS - 1) / PG::IDS;    // id registers per row
};

// (the members are what walk_steps wants, see dual_walk.h)
template <int D, bool ZB, int R> struct TripleStep {
    using C = TripleCfg<D, ZB, R>;
    using PG = typename C::PG;
    static constexpr int NIDS = R * C::IDR, N = PG::N, EPI = PG::EPI, LDS_FLOATS = C::LDS_FLOATS;

    static __device__ __forceinline__ void init(float *lds, int lane) {
        static_assert(PG::ZERO_FLOATS <= 64, "one store a lane");
        if (lane < PG::ZERO_FLOATS) lds[C::OFF_ZERO + lane] = 0.f;
        wave_sync();
    }
    static __device__ __forceinline__ int id_entry(int lane, int r) { return EPI * PG::IDS * r + PG::id_entry(lane, PG::IDS); }
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
        const int (&k)[4] = d.k;
        int kmax = 0;
#pragma unroll
        for (int p = 0; p < R; ++p) kmax = k[p] > kmax ? k[p] : kmax;

        // ---- 1. gather and the tiles of S
        floatx4 z[C::DEPTH][3][N];
        const char *zlane = (const char *)Z + 16 * (opaque_tid() % PG::LPR);
        auto load = [&](auto uu) {
            constexpr int unit = decltype(uu)::value, p = unit / C::NCH, h = unit % C::NCH;
            static_for<0, 3>([&](auto tt) {
                static_for<0, N>([&](auto ss) {
                    constexpr int t = decltype(tt)::value, s = decltype(ss)::value, n = t * N + s;
                    if (t < 2 || 32 + s * EPI < k[p]) {  // the first two tiles are full
                        const int32_t id = PG::template bcast_id<n % PG::IDS>(idv[C::IDR * p + n / PG::IDS]);
                        z[unit % C::DEPTH][t][s] = *(const floatx4 *)(zlane + (int64_t)id * C::RB + h * C::CB);
                    }
                });
            });
        };
        static_for<0, C::DEPTH>(load);
        loaded();
        const int lane = opaque_tid();  // after the loads: what derives from it is not kept across them
        const int a = lane & 15, q = lane >> 4;                 // MFMA view: entry a of a tile, column group q
        const int g = R == 4 ? lane >> 4 : 0, i = lane & 15;    // solver view: system g, lane i of its group
        float y0, y1 = 0.f, y2 = 0.f;  // labels of the entries i, 16 + i and 32 + i of this lane's system; R = 1: y0 of entry `lane`
        if constexpr (R == 1) {
            y0 = lane < k[0] ? (values ? values[d.b[0] + lane] : 1.f) : 0.f;
        } else {
            int myk = 0;
            int64_t myb = 0;
#pragma unroll
            for (int p = 0; p < R; ++p) {
                myk = g == p ? k[p] : myk;
                myb = g == p ? d.b[p] : myb;
            }
            y0 = i < myk ? 1.f : 0.f;
            y1 = 16 + i < myk ? 1.f : 0.f;
            y2 = 32 + i < myk ? 1.f : 0.f;
            if (values) {
                int at = i;
                asm volatile("" : "+v"(at));  // no zero-extended copy of i across the step
                if (i < myk) y0 = values[myb + at];
                if (16 + i < myk) y1 = values[myb + at + 16];
                if (32 + i < myk) y2 = values[myb + at + 32];
            }
        }
        {
            int32_t *idl = (int32_t *)(lds + C::OFF_ID);
#pragma unroll
            for (int n = 0; n < NIDS; ++n) idl[n / C::IDR * C::KS + id_entry(lane, n % C::IDR)] = idv[n];
        }
        float *mfma_at = lds + tile_block(a, q);  // MFMA view: row a, columns 4 q .. of the first system's tile
        char *stage = (char *)(lds + C::OFF_10);
        floatx4 c10[R], c20[R], c11[R], c21[R], c22[R];  // cij[p][v] = S_ij[a][4 q + v]
        static_for<0, R>([&](auto pp) {
            constexpr int p = decltype(pp)::value;
            const floatx4 zero4 = floatx4{0.f, 0.f, 0.f, 0.f};
            floatx4 c00 = zero4;
            c10[p] = c20[p] = c11[p] = c21[p] = c22[p] = zero4;
            static_for<0, C::NCH>([&](auto hh) {
                constexpr int unit = p * C::NCH + decltype(hh)::value;
                // what derives from the lane is formed again for each unit rather than kept
                const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;
                const int put = PG::put_base(lane), get = PG::get_base(a, q);
                static_for<0, 3>([&](auto tt) {
                    static_for<0, N>([&](auto ss) {
                        constexpr int t = decltype(tt)::value, s = decltype(ss)::value;
                        if (t < 2 || 32 + s * EPI < k[p])
                            *(floatx4 *)(stage + t * 16 * C::CB + PG::template put_at<s>(put)) = z[unit % C::DEPTH][t][s];
                    });
                });
                wave_sync();
                if constexpr (unit + C::DEPTH < C::UNITS) load(std::integral_constant<int, unit + C::DEPTH>{});
                const bool have = 32 + a < k[p];  // slots of the third tile beyond the row's k read zeros
                const char *const zero = (const char *)(lds + C::OFF_ZERO);
                auto piece = [&](int t, int j) {
                    const char *at = stage + t * 16 * C::CB + (j & 1 ? get ^ 64 : get);
                    return (t < 2 || have ? at : zero) + 128 * (j >> 1);
                };
                __builtin_amdgcn_s_setprio(1);  // matrix-core work first: other wavefronts fill in with vector work
#pragma unroll
                for (int j = 0; j < N; j += ZB ? 1 : 2) {
                    auto operand = [&](int t) {
                        if constexpr (ZB) return *(const bf16x8 *)piece(t, j);
                        else return split_operand(*(const float4 *)piece(t, j), *(const float4 *)piece(t, j + 1));
                    };
                    const auto o0 = operand(0), o1 = operand(1), o2 = operand(2);
                    auto product = [&](const auto &x, const auto &y, floatx4 &acc) {
                        if constexpr (ZB) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc, 0, 0, 0);
                        else acc = split_mfma(x, y, acc);
                    };
                    product(o0, o0, c00);
                    product(o0, o1, c10[p]);
                    product(o0, o2, c20[p]);
                    product(o1, o1, c11[p]);
                    product(o1, o2, c21[p]);
                    product(o2, o2, c22[p]);
                }
                __builtin_amdgcn_s_setprio(0);
                wave_sync();  // the next unit reuses the stage
            });
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float one = 4 * q + v == a ? 1.f : 0.f;
                c00[v] += one;
                c11[p][v] += one;
                c22[p][v] += one;
            }
            *(floatx4 *)(mfma_at + C::OFF_T + p * TILE_FLOATS) = c00;
        });
        between();
        // the second gather (step 4): the rows advance together, EPL entries per lane and round; the first round's entries are on their way
        // while the systems are solved, the others two rounds ahead
        constexpr int LPR = C::RB / 16, EPI2 = 64 / LPR, EPL = 4, EPR = EPL * EPI2, NV = ZB ? 2 : 1;
        constexpr int ROUNDS = (48 + EPR - 1) / EPR, BUFS = ROUNDS < 3 ? ROUNDS : 3;
        const int32_t *ids = (const int32_t *)(lds + C::OFF_ID);
        floatx4 zz[BUFS][R][EPL];
        auto again = [&](auto rr) {  // padded entries have t = 0 and the id of the row's first entry
            constexpr int r = decltype(rr)::value;
            const int lane = opaque_tid();
            const char *col = (const char *)Z + 16 * (lane % LPR);
            int4 id[R];
#pragma unroll
            for (int p = 0; p < R; ++p) id[p] = *(const int4 *)(ids + p * C::KS + r * EPR + EPL * (lane / LPR));
#pragma unroll
            for (int p = 0; p < R; ++p)
                if (r * EPR < k[p]) {  // uniform
                    const int at[EPL] = {id[p].x, id[p].y, id[p].z, id[p].w};
#pragma unroll
                    for (int x = 0; x < EPL; ++x) zz[r % BUFS][p][x] = *(const floatx4 *)(col + (int64_t)at[x] * C::RB);
                }
        };
        if constexpr (R == 4) again(std::integral_constant<int, 0>{});
        auto put_tiles = [&](int off, const floatx4 (&c)[R]) {
#pragma unroll
            for (int p = 0; p < R; ++p) *(floatx4 *)(mfma_at + off + p * TILE_FLOATS) = c[p];
        };
        put_tiles(C::OFF_10, c10);
        put_tiles(C::OFF_20, c20);
        wave_sync();

        // ---- 2. elimination, a block column at a time
        float *row_at = lds + g * TILE_FLOATS + 16 * i;  // solver view: row i of system g
        const int swz = (i >> 1 & 3) << 2;               // block b of that row lies at row_at + (4 b ^ swz)
        auto put_row = [&](int off, const float (&s)[16]) {
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4)
                *(float4 *)(row_at + off + (4 * c4 ^ swz)) = make_float4(s[4 * c4], s[4 * c4 + 1], s[4 * c4 + 2], s[4 * c4 + 3]);
        };
        float s0[16], s1[16], s2[16], ri0 = 1.f, ri1 = 1.f, ri2 = 1.f;
        bool bad = false;
        // R = 1: the rows of the first block column over the groups 0, 1 and 2, those of the second over the halves of the wavefront
        float *one_at = lds + 16 * i;
        if constexpr (R == 1) load_tile_row(one_at + (q == 3 ? 0 : q) * C::AREA, i, s0);  // S_00, S_10, S_20
        else {
            load_tile_row(row_at + C::OFF_T, i, s0);
            load_tile_row(row_at + C::OFF_10, i, s1);
            load_tile_row(row_at + C::OFF_20, i, s2);
        }
        dpp_settle(s0[0]);
        static_for<0, 16>([&](auto ci) {
            if constexpr (R == 1) eliminate_shared<decltype(ci)::value, 16>(s0, y0, ri0, lane, bad);
            else eliminate_column<decltype(ci)::value>(s0, y0, ri0, i, bad, RowBelow{s1, y1}, RowBelow{s2, y2});
        });
        wave_sync();  // every lane has read its rows
        if constexpr (R == 1) {
            if (q == 1 || q == 2) put_row(q == 1 ? C::OFF_T : C::OFF_21, s0);
            y1 = from_lane_row<1>(y0);
            y2 = from_lane_row<2>(y0);
        } else {
            put_row(C::OFF_T, s1);
            put_row(C::OFF_21, s2);
        }
        wave_sync();
#pragma unroll
        for (int p = 0; p < R; ++p) {
            // lane (a, q) supplies L_i[a][4 q + e] to instruction e on both sides: the contraction runs over all 16 columns
            const floatx4 l1 = *(const floatx4 *)(mfma_at + C::OFF_T + p * TILE_FLOATS), l2 = *(const floatx4 *)(mfma_at + C::OFF_21 + p * TILE_FLOATS);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                c11[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(-l1[e], l1[e], c11[p], 0, 0, 0);
                c21[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(-l1[e], l2[e], c21[p], 0, 0, 0);
                c22[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(-l2[e], l2[e], c22[p], 0, 0, 0);
            }
        }
        wave_sync();
        put_tiles(C::OFF_T, c11);
        put_tiles(C::OFF_21, c21);
        wave_sync();
        if constexpr (R == 1) {
            load_tile_row(one_at + (q < 2 ? C::OFF_T : C::OFF_21), i, s1);
            y1 = q < 2 ? y1 : y2;
        } else {
            load_tile_row(row_at + C::OFF_T, i, s1);
            load_tile_row(row_at + C::OFF_21, i, s2);
        }
        dpp_settle(s1[0]);
        static_for<0, 16>([&](auto ci) {
            if constexpr (R == 1) eliminate_shared<decltype(ci)::value, 32>(s1, y1, ri1, lane, bad);
            else eliminate_column<decltype(ci)::value>(s1, y1, ri1, i, bad, RowBelow{s2, y2});
        });
        wave_sync();
        if constexpr (R == 1) {
            if (q == 2) put_row(C::OFF_T, s1);
            y2 = from_lane_row<2>(y1);
        } else {
            put_row(C::OFF_T, s2);
        }
        wave_sync();
#pragma unroll
        for (int p = 0; p < R; ++p) {
            const floatx4 l2 = *(const floatx4 *)(mfma_at + C::OFF_T + p * TILE_FLOATS);
#pragma unroll
            for (int e = 0; e < 4; ++e) c22[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(-l2[e], l2[e], c22[p], 0, 0, 0);
        }
        wave_sync();
        put_tiles(C::OFF_T, c22);
        wave_sync();
        load_tile_row(row_at + C::OFF_T, i, s2);
        dpp_settle(s2[0]);
        static_for<0, 16>([&](auto ci) {
            constexpr int c = decltype(ci)::value;
            if (32 + c < kmax) eliminate_column<c>(s2, y2, ri2, i, bad);  // beyond every row's k: identity rows
        });
        // a row past the end of the list stands for the step's first entry many times over: its pivots mean nothing
        int rel = d.row.rel[0];
        if constexpr (R == 4) {
            const int rel_lo = g & 1 ? d.row.rel[1] : d.row.rel[0], rel_hi = g & 1 ? d.row.rel[3] : d.row.rel[2];
            rel = g & 2 ? rel_hi : rel_lo;
        }
        if (bad && rel >= 0) atomicOr(err_flag, 1);

        // ---- 3. t of the three blocks, backwards
        float za = 0.f, zb = 0.f;
        auto add_columns = [&](int off, float &t) {  // += S_ij^T t: column i of the tile at `off`, t of the rows through DPP
            float bt[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) bt[m] = lds[off + g * TILE_FLOATS + 16 * m + (((i >> 2) ^ (m >> 1) & 3) << 2) + (i & 3)];
            dpp_settle(t);
            static_for<0, 8>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                fmac_bcast16<2 * m>(za, t, bt[2 * m]);
                fmac_bcast16<2 * m + 1>(zb, t, bt[2 * m + 1]);
            });
        };
        auto row_operations = [&](const float (&s)[16]) {
            za += zb;
            static_for<0, 16>([&](auto ci) {
                constexpr int c = decltype(ci)::value;
                dpp_settle(za);
                fmac_bcast16_neg<c>(za, za, s[c]);
            });
        };
        float t2 = y2 * ri2 * ri2;
        add_columns(C::OFF_21, t2);
        row_operations(s1);
        float t1 = (y1 - za) * ri1 * ri1;
        za = zb = 0.f;
        add_columns(C::OFF_20, t2);
        add_columns(C::OFF_10, t1);
        row_operations(s0);
        const float t0 = (y0 - za) * ri0 * ri0;
        wave_sync();  // every lane has read its row of S_22
        float *tbuf = lds + C::OFF_T;
        if (R == 4 || q == 0) {  // R = 1: t0 is that of the first group, which holds the rows of S_00
            tbuf[g * C::KS + i] = t0;
            tbuf[g * C::KS + 16 + i] = t1;
            tbuf[g * C::KS + 32 + i] = t2;
            tbuf[g * C::KS + 48 + i] = 0.f;
        }
        wave_sync();

        // ---- 4. r = Z_I^T t
        static_for<R == 4 ? 1 : 0, BUFS>(again);
        floatx4 rv[R][NV];
#pragma unroll
        for (int p = 0; p < R; ++p)
#pragma unroll
            for (int n = 0; n < NV; ++n) rv[p][n] = floatx4{0.f, 0.f, 0.f, 0.f};
        static_for<0, ROUNDS>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
#pragma unroll
            for (int p = 0; p < R; ++p)
                if (r * EPR < k[p]) {
                    const float4 te = *(const float4 *)(tbuf + p * C::KS + r * EPR + EPL * (lane / LPR));
                    const float t[EPL] = {te.x, te.y, te.z, te.w};
#pragma unroll
                    for (int x = 0; x < EPL; ++x)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float w = zz[r % BUFS][p][x][c];
                            if constexpr (ZB) {
                                rv[p][c / 2][2 * (c & 1)] += t[x] * __uint_as_float(__float_as_uint(w) << 16);
                                rv[p][c / 2][2 * (c & 1) + 1] += t[x] * __uint_as_float(__float_as_uint(w) & 0xffff0000u);
                            } else {
                                rv[p][0][c] += t[x] * w;
                            }
                        }
                }
            if constexpr (r + BUFS < ROUNDS) again(std::integral_constant<int, r + BUFS>{});
        });
        last();
        if constexpr (R == 1) out.template store_one<LPR>(rv[0], lane);
        else out.template store<LPR>(rv, lane);
    }
};

// One row (list item `item`) by one wavefront.
template <int D, bool ZB>
__device__ __forceinline__ void dual_triple_row(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                const float *__restrict__ values, const void *__restrict__ Z, float *__restrict__ R,
                                                int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                int32_t *__restrict__ err_flag, int item, float *lds) {
    using S = TripleStep<D, ZB, 1>;
    S::init(lds, opaque_tid());
    const int32_t rel = list[item];
    const int64_t b = indptr[r0 + rel];
    const RowsDesc d = {{{rel, -1, -1, -1}}, {b, b, b, b}, {(int)(indptr[r0 + rel + 1] - b), 0, 0, 0}};
    int32_t idv[S::NIDS];
    S::ids(indices, d, opaque_tid(), idv);
    S::solve(values, Z, err_flag, lds, d, idv, [] {}, [] {}, [] {}, RowsOut{R + r0 * ldr, ldr, d.row});
}

}  // namespace als
