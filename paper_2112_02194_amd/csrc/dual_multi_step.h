// Dual row update for rows with 16 < k <= 32 stored entries.  The algebra is in the header comment of
// dual_prepare.hip.
#pragma once

#include "dual_common.h"

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
//   5. r = Z_I^T t: bf16 Z from the tiles in registers on the matrix cores; fp32 Z with one lane per group
//      of four output columns, gathering the entries a second time.
// What bounds it: bf16 Z (50M power-law rows): the instructions of two wavefronts per SIMD, one every five clocks each, and
// the latency of the gather; fp32 Z whose rows meet in the caches: the address unit, which takes a clock per lane of the
// first gather (sixteen rows per instruction, 64 clocks), 94% busy on 10M pages of locality.
// Against an elimination of all 32 columns with a triangular back-substitution through LDS (616 multiply-adds with a DPP
// operand, 392 here; LDS accesses of 4 bytes with a select each, 16 bytes here; 3 219 instructions per step, 2 373 here) a
// half of the power-law rows (d = 128, bf16) takes 41.4 instead of 44.6 ms and one of 10M pages (d = 128, fp32) 7.50 instead
// of 7.65 ms, the latter 7.15 ms with the 16-byte loads of the second gather; 1M x 1M, d = 64: 705 -> 671 us.

// LDS of one wavefront: two regions of four 16 x 16 tiles (P: A, then L, then C, then t; Q: B), one per system.
struct MultiCfg {
    static constexpr int K = 32, TILE = TILE_FLOATS, REGION = 4 * TILE;
    static constexpr int OFF_P = 0, OFF_Q = REGION, OFF_ID = 2 * REGION;
    static constexpr int LDS_FLOATS = OFF_ID + 4 * K;  // ids of the second gather
    // bf16 Z: t cut into three bf16 parts plus a block of zeros, [4][4 rows][K], and the lanes' dump slots in P; the
    // finished rows of r in Q
    static constexpr int LDS_FLOATS_RESIDENT = 2 * REGION;
    static_assert(REGION >= 16 * K + 64 && REGION >= 4 * 128, "P and Q hold what step 5 stages");
};
// bf16 Z: the gathered tiles stay in registers (4 rows x 2 tiles x D/32 operands of four registers) until r = Z_I^T t is
// formed from them on the matrix cores, so nothing is gathered twice.
template <bool ZB> constexpr bool multi_resident() { return ZB; }

// One step: the four rows list[4 blk .. 4 blk + 3] (blk * 4 < count).
template <int D, bool ZB>
__device__ __forceinline__ void dual_multi_step(const int64_t *__restrict__ indptr,
                                                const int32_t *__restrict__ indices,
                                                const float *__restrict__ values, const void *__restrict__ Z,
                                                float *__restrict__ R, int64_t ldr, int64_t r0,
                                                const int32_t *__restrict__ list, int count,
                                                int32_t *__restrict__ err_flag, int blk, float *lds) {
    using C = MultiCfg;
    constexpr int K = C::K, NJ = z_pieces<D, ZB>(), CPL = D >= 128 ? 2 : 1;
    constexpr bool RES = multi_resident<ZB>();
    int32_t *ids = (int32_t *)(lds + C::OFF_ID);
    const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;  // MFMA view: entry a of a tile, column group q
    const int g = lane >> 4, i = lane & 15;                         // solver view: system g, lane i of its group
    float *mfma_at = lds + tile_block(a, q);        // MFMA view: row a, columns 4 q .. of the first system's tile
    float *row_at = lds + g * C::TILE + 16 * i;     // solver view: row i of system g
    const int swz = (i >> 1 & 3) << 2;              // block b of that row lies at row_at + (4 b ^ swz)

    // Row descriptors of all four rows first (one 16-byte read of the list entries - the list's workspace is
    // padded for it; past the end of the list the first entry stands in - then the four indptr pairs
    // together): one wait per stage instead of one per row.
    int64_t u[4], b[4], b1[4];
    int k[4], kmax = 0, rel[4];
    {
        const ListQuad r4 = *(const ListQuad *)(list + (int64_t)blk * 4);
        const int first = blk * 4;
        rel[0] = r4.x;
        rel[1] = first + 1 < count ? r4.y : r4.x;
        rel[2] = first + 2 < count ? r4.z : r4.x;
        rel[3] = first + 3 < count ? r4.w : r4.x;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        b[p] = indptr[r0 + rel[p]];
        b1[p] = indptr[r0 + rel[p] + 1];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const bool have = blk * 4 + p < count;
        u[p] = have ? r0 + rel[p] : -1;  // past the end of the list: the step's first row once more, not stored
        k[p] = (int)(b1[p] - b[p]);
        kmax = k[p] > kmax ? k[p] : kmax;
    }

    // ---- 1. the tiles of S
    // the column ids of all four rows first: one wait, not one per row.  A slot past the row's k holds the id of
    // the row's first entry with the top bit set: no load for the products, and a harmless, in-range row of the
    // row's own for the second gather (where such a slot meets t = 0)
    int32_t idv[4][2];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int e = 16 * t + a;
            const int32_t id = indices[b[p] + (e < k[p] ? e : 0)];  // clamped: unconditional load
            idv[p][t] = e < k[p] ? id : (id | (int32_t)0x80000000);
        }
    // labels of the entries i and 16 + i of this lane's system (the class has more than 16 entries per row)
    float y0 = 1.f, y1 = 0.f;
    {
        int myk = 0;
        int64_t myb = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            myk = g == p ? k[p] : myk;
            myb = g == p ? b[p] : myb;
        }
        if (16 + i < myk) y1 = 1.f;
        if (values) {
            y0 = values[myb + i];
            if (16 + i < myk) y1 = values[myb + 16 + i];
        }
    }
    float4 zkeep[RES ? 4 : 1][2][NJ];
    floatx4 cc[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float4 zrow[2][NJ];
        float4 (&z)[2][NJ] = RES ? zkeep[RES ? p : 0] : zrow;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int32_t id = idv[p][t];
            if (!RES && q == 0) ids[p * K + 16 * t + a] = id & 0x7fffffff;
            if (t == 0) {  // every row of the class has more than 16 entries: this tile is full
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[t][j] = load_piece<D, ZB>(Z, id & 0x7fffffff, j, q);
            } else {
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[t][j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (id >= 0) {  // one masked region per tile, not one per load
#pragma unroll
                    for (int j = 0; j < NJ; ++j) z[t][j] = load_piece<D, ZB>(Z, id, j, q);
                }
            }
        }
        TileOperand<D, ZB> op[2];
        op[0].set(z[0]);
        op[1].set(z[1]);
        __builtin_amdgcn_s_setprio(1);  // matrix-core work first: other wavefronts fill in with vector work
        const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
        floatx4 ca = tile_product<D, ZB>(op[0], op[0], zero);
        const floatx4 cb = tile_product<D, ZB>(op[0], op[1], zero);
        cc[p] = tile_product<D, ZB>(op[1], op[1], zero);
        // ca[v] = A[a][4 q + v], cb[v] = B[a][4 q + v], cc[p][v] = C[a][4 q + v] (A and C are symmetric)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float one = 4 * q + v == a ? 1.f : 0.f;
            ca[v] += one;
            cc[p][v] += one;
        }
        *(floatx4 *)(mfma_at + C::OFF_P + p * C::TILE) = ca;
        *(floatx4 *)(mfma_at + C::OFF_Q + p * C::TILE) = cb;
        __builtin_amdgcn_s_setprio(0);
    }
    wave_sync();

    // ---- 2. elimination of the columns of A
    float s0[16], s1[16], ri0 = 1.f, ri1 = 1.f;
    bool bad = false;
    load_tile_row(row_at + C::OFF_P, i, s0);
    load_tile_row(row_at + C::OFF_Q, i, s1);
    dpp_settle(s0[0]);
    static_for<0, 16>([&](auto ci) { eliminate_column<decltype(ci)::value, true>(s0, s1, y0, y1, ri0, i, bad); });

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
        float none = 0.f;
        if (16 + c < kmax) eliminate_column<c, false>(s1, s1, y1, none, ri1, i, bad);  // beyond every row's k: identity rows
    });
    if (bad) atomicOr(err_flag, 1);

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
    if constexpr (RES) {
        // ---- 5. r = Z_I^T t from the tiles in registers (zt_times_t, dual_common.h); parts[x][row][e]: part
        // x of t, x = 3 a block of zeros; the finished rows are staged for 8-byte stores
        float *parts = lds + C::OFF_P, *dump = parts + 16 * K + lane;
        wave_sync();  // every lane has read its rows of C and its column of B
#pragma unroll
        for (int bk = 0; bk < 2; ++bk) {
            float x1, x2;
            const float t = bk ? t1 : t0;
            t_parts(t, x1, x2);
            const int e = g * K + 16 * bk + i;
            parts[e] = t;
            parts[4 * K + e] = x1;
            parts[8 * K + e] = x2;
            parts[12 * K + e] = 0.f;
        }
        const SelOperands sel = make_sel(lane);
        wave_sync();
        const float *mine = parts + (a < 3 ? a : 3) * 4 * K + 4 * q;
        float *rbuf = lds + C::OFF_Q;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const bf16x8 top[1] = {t_operand(mine + p * K, true)};
            floatx4 out[2 * NJ];
#pragma unroll
            for (int x = 0; x < 2 * NJ; ++x) out[x] = floatx4{0.f, 0.f, 0.f, 0.f};
            zt_times_t<2, NJ>([&](int tt, int j) { return __builtin_bit_cast(bf16x8, zkeep[RES ? p : 0][tt][j]); }, top, sel, out);
#pragma unroll
            for (int x = 0; x < 2 * NJ; ++x)
                *(q == 0 ? rbuf + p * D + column_of_result(x >> 1, x & 1, a) : dump) = out[x][0] + out[x][1] + out[x][2];
        }
        wave_sync();
        const bool col_ok = lane * CPL < D;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (u[p] >= 0 && col_ok) {
                if constexpr (CPL == 2) *(float2 *)(R + u[p] * ldr + 2 * lane) = *(const float2 *)(rbuf + p * D + 2 * lane);
                else R[u[p] * ldr + lane] = rbuf[p * D + lane];
            }
        }
        return;
    }
    float *tbuf = lds + C::OFF_P;
    wave_sync();  // every lane has read its row of C
    tbuf[g * K + i] = t0;
    tbuf[g * K + 16 + i] = t1;
    wave_sync();

    // ---- 5. r = Z_I^T t (second gather of the row's entries): 16 bytes of an entry per lane, so that one instruction takes
    // GatherCols<D>::EPI entries; the four rows advance together, EPL entries per lane and round.  Per round: first the
    // ids and t of all rows from LDS, then the loads, then the products - no wait and no lane-dependent branch between
    // two loads.
    {
        using GC = GatherCols<D>;
        constexpr int EPL = 2, EPR = EPL * GC::EPI;
        const int mine = EPL * (lane / GC::LPR);
        const float *col = (const float *)Z + 4 * (lane % GC::LPR);
        floatx4 rv[4][1];
#pragma unroll
        for (int p = 0; p < 4; ++p) rv[p][0] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int e0 = 0; e0 < kmax; e0 += EPR) {  // padded entries have t = 0 and the id of the row's first entry
            int2 id[4];
            float2 te[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                id[p] = *(const int2 *)(ids + p * K + e0 + mine);
                te[p] = *(const float2 *)(tbuf + p * K + e0 + mine);
            }
            floatx4 zz[4][EPL];
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (e0 < k[p]) {  // uniform
                    zz[p][0] = *(const floatx4 *)(col + (int64_t)id[p].x * D);
                    zz[p][1] = *(const floatx4 *)(col + (int64_t)id[p].y * D);
                }
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (e0 < k[p]) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        rv[p][0][c] += te[p].x * zz[p][0][c];
                        rv[p][0][c] += te[p].y * zz[p][1][c];
                    }
                }
        }
        store_rows<GC::LPR>(rv, R, ldr, u, lane);
    }
}

}  // namespace als
