// Dual row update for 48 < k <= 128 (d = 128; k <= 64 also at d = 64), in classes KT = 4..8 (k <= 16*KT); under conjugate
// gradients for all rows, those of up to 48 entries with KT = 3.  The algebra is in the header comment of dual_prepare.hip.
#pragma once

#include "dual_common.h"
#include "tri_cg.h"
#include "tri_solve.h"

namespace als {

// One wavefront per row with k <= K = 16*KT entries (KT = 3..8).
//   1. S = I + Z_I Z_I^T tile by tile, into a lower triangle in LDS.  The first wide_tiles() tiles of sixteen entries are
//      loaded together and stay in registers as operands; the last one (fp32, k > 80) is loaded when it is needed.  Where
//      wide_staged(), side-by-side lanes load side-by-side pieces of a row (PieceGather, dual_common.h), and the tiles go
//      through the triangle's place in LDS into the operand layout.
//   2./3. Block elimination S = M P M^T and back-substitution by the wavefront (tri_solve.h).
//   4. r = Z_I^T t: with bf16 Z from the tiles still in registers, on the matrix cores (zt_times_t,
//      dual_common.h: bf16 entries are exact operands); with fp32 Z with four adjacent output columns per lane,
//      gathering the entries a second time (the hi + lo operands kept for S carry z only to 2^-16, which is
//      enough for S = I + Z Z^T but would show in r).
template <int D, int KT, bool ZB> constexpr bool wide_resident() { return ZB; }

// Tiles that stay in registers.  fp32, d = 128: a tile takes 32 registers as loaded and 32 as operands.  From KT = 6 on the last tile, which is
// needed last, is loaded then; among the first it left the compiler no registers, which then waited for its eight loads one by
// one (200 000 rows of 100 / 120 entries 5.23 / 6.72 ms, as it is 4.86 / 5.91; another tile fewer 4.86 / 6.12; with four resident 6.00 / 7.36).
template <int KT, bool ZB> constexpr int wide_tiles() { return ZB || KT < 6 ? KT : KT - 1; }
// Long rows of Z only.  10M pages with host locality (d = 128, fp32), KT = 4 .. 8, ms per epoch, straight into the operand
// layout / staged: 4.25 / 4.07, 2.98 / 2.91, 2.35 / 2.12, 1.93 / 1.86, 1.24 / 1.16.  Shorter rows lose (measured with the direct
// solver's KT = 3, which dual_triple_step.h has replaced): 1M x 1M (d = 64) 1.22 / 1.26 ms, 300k bf16 rows (d = 128) 76 / 81 us.
template <int D, bool ZB> constexpr bool wide_staged() { return D == 128 && !ZB; }

template <int D, int KT> struct WideCfg {
    static constexpr int K = 16 * KT;
    static constexpr int TRI = tri_row<K>(K);           // lower triangle, rows padded (tri_solve.h)
    static constexpr int OFF_COL = TRI;              // solver's auxiliary buffer
    static constexpr int OFF_T = OFF_COL + TRI_AUX_FLOATS<K>;  // tbuf[K]
    static constexpr int OFF_ID = OFF_T + K;         // ids[K]
    static constexpr int STAGE_FLOATS = wide_staged<D, false>() ? RowGather<D, false>::STAGE_FLOATS : 0;  // over everything else, before anything is there
    static constexpr int LDS_FLOATS = OFF_ID + K > STAGE_FLOATS ? OFF_ID + K : STAGE_FLOATS;
};

// CG: the k x k system is solved by conjugate gradients (tri_cg.h) instead of the panel elimination.
template <int D, int KT, bool ZB, bool CG>
__device__ __forceinline__ void dual_wide_step(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                               const float *__restrict__ values, const void *__restrict__ Z,
                                               float *__restrict__ R, int64_t ldr, int64_t r0,
                                               const int32_t *__restrict__ list, int32_t *__restrict__ err_flag,
                                               int item, float *lds, int cg_iters, float cg_tol) {
    using C = WideCfg<D, KT>;
    constexpr int K = C::K, NJ = z_pieces<D, ZB>();
    constexpr bool RES = wide_resident<D, KT, ZB>();
    float *tri = lds, *aux = lds + C::OFF_COL, *tbuf = lds + C::OFF_T;
    int32_t *ids = (int32_t *)(lds + C::OFF_ID);
    const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;
    const int64_t u = r0 + list[item];
    const int64_t b = indptr[u];
    const int k = (int)(indptr[u + 1] - b);  // <= K by the list's class

    // ---- 1. S tiles
    // With the direct solver the class holds rows with more than 16 (KT - 1) entries only: all tiles but the last are full
    // (under CG shorter rows come through the same kernel).  A slot past k has the id of the row's first entry (and meets t = 0
    // below); its operand is zero.
    using RG = RowGather<D, ZB>;
    constexpr bool STAGED = wide_staged<D, ZB>();
    constexpr int RT = wide_tiles<KT, ZB>(), N = RG::N, T0 = STAGED ? RT : 0;  // tiles from T0 on are loaded in operand layout
    static_assert(N == NJ, "as many registers as loaded and as operand");
    typedef TileOperand<D, ZB> Op;
    int32_t idv[STAGED ? RT : 1], myid[T0 < KT ? KT - T0 : 1];
    const int in_tile = RG::id_entry(lane);
#pragma unroll
    for (int t = 0; t < T0; ++t) {
        const int e = 16 * t + in_tile;
        idv[t] = indices[b + (e < k ? e : 0)];
    }
#pragma unroll
    for (int t = T0; t < KT; ++t) {
        const int e = 16 * t + a;
        const int32_t id = indices[b + (e < k ? e : 0)];
        myid[t - T0] = e < k ? id : (id | (int32_t)0x80000000);  // a padded slot: negative, and still a row of the table
        if (!RES && q == 0) ids[e] = id;  // beyond what a stage takes, where there are such tiles
    }
    auto fetch = [&](int t, float4 (&raw)[NJ]) {  // t >= T0
        const int32_t id = myid[t < T0 ? 0 : t - T0];
        if (!CG && t < KT - 1) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) raw[j] = load_piece<D, ZB>(Z, id & 0x7fffffff, j, q);
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j) raw[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (id >= 0) {  // one masked region per tile, not one per load
#pragma unroll
                for (int j = 0; j < NJ; ++j) raw[j] = load_piece<D, ZB>(Z, id, j, q);
            }
        }
    };
    Op zop[RT];
    if constexpr (STAGED) {
        static_assert(KT == RT || C::OFF_ID >= C::STAGE_FLOATS, "ids of tiles beyond the staged ones are in LDS already");
        floatx4 raw[RT][N];  // (the plain vector type: as float4 they are copied by way of scratch memory)
        const char *zlane = (const char *)Z + 16 * (lane % RG::LPR);
        // Under CG the smallest instance takes rows from one entry on: instructions that only meet slots beyond the row's k are left out
        // (60 000 rows of 1 / 13 entries, d = 128, the call: 220 / 337 us with them, 192 / 321 without).
        constexpr bool SHORT = CG && KT == 3;
        static_for<0, RT * N>([&](auto ii) {
            constexpr int t = decltype(ii)::value / N, s = decltype(ii)::value % N;
            if (!SHORT || 16 * t + RG::EPI * s < k)
                raw[t][s] = *(const floatx4 *)(zlane + (int64_t)RG::template bcast_id<s>(idv[t]) * RG::RB);
        });
        char *stage = (char *)lds;
        const int put = RG::put_base(lane), get = RG::get_base(a, q);
        static_for<0, RT>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            static_for<0, N>([&](auto ss) {
                constexpr int s = decltype(ss)::value;
                if (!SHORT || 16 * t + RG::EPI * s < k) *(floatx4 *)(stage + RG::template put_at<s>(put)) = raw[t][s];
            });
            wave_sync();
            const bool have = 16 * t + a < k;
            float4 o[NJ];
            static_for<0, NJ>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                float4 x = *(const float4 *)(stage + (j & 1 ? get ^ 64 : get) + 128 * (j >> 1));
                if constexpr (CG || t == KT - 1) x = make_float4(have ? x.x : 0.f, have ? x.y : 0.f, have ? x.z : 0.f, have ? x.w : 0.f);
                o[j] = x;
            });
            zop[t].set(o);
            wave_sync();  // the next tile, or the triangle, takes the place
        });
#pragma unroll
        for (int t = 0; t < RT; ++t) ids[16 * t + in_tile] = idv[t];  // several lanes, the same value
    } else {
        float4 raw[RT][NJ];
#pragma unroll
        for (int t = 0; t < RT; ++t) fetch(t, raw[t]);
#pragma unroll
        for (int t = 0; t < RT; ++t) zop[t].set(raw[t]);
    }
#pragma unroll
    for (int t1 = 0; t1 < KT; ++t1) {
        Op zb;
        if (t1 < RT) {
            zb = zop[t1 < RT ? t1 : 0];
        } else {
            float4 raw[NJ];
            fetch(t1, raw);
            zb.set(raw);
        }
#pragma unroll
        for (int t2 = 0; t2 <= t1; ++t2) {
            floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
            if (t2 == t1) {
                acc = tile_product<D, ZB>(zb, zb, acc);
            } else if (t2 < RT) {
                acc = tile_product<D, ZB>(zop[t2 < RT ? t2 : 0], zb, acc);
            } else {
                float4 raw[NJ];
                fetch(t2, raw);
                Op za;
                za.set(raw);
                acc = tile_product<D, ZB>(za, zb, acc);
            }
            // acc[v] = S[Rr][c], Rr = 16*t1 + a, c = 16*t2 + 4q + v (S is symmetric).  The triangle's rows are
            // padded to whole tiles, so a diagonal tile is stored whole: what lies beyond the diagonal lands in
            // the row's padding
            const int Rr = 16 * t1 + a, c0 = 16 * t2 + 4 * q;
            if (t2 == t1) {  // known after unrolling: the identity only meets diagonal tiles
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] += c0 + v == Rr ? 1.f : 0.f;
            }
            *(float4 *)(tri + tri_row<K>(Rr) + c0) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
    }
    wave_sync();

    // ---- 2./3. elimination and back-substitution (tri_solve.h); lane i holds the labels of entries i, 64+i
    {
        float y0 = 0.f, y1 = 0.f;
        if (lane < k) y0 = values ? values[b + lane] : 1.f;
        if (64 + lane < k) y1 = values ? values[b + 64 + lane] : 1.f;
        if constexpr (CG) tri_cg<K>(tri, aux, tbuf, y0, y1, k, cg_iters, cg_tol);
        else tri_solve<K>(tri, aux, tbuf, y0, y1, k, err_flag);
    }

    // ---- 4. r = Z_I^T t
    if constexpr (RES) {
        // the triangle is free now: the remainders of the cut of t, a block of zeros and the finished row go there
        static_assert(tri_row<K>(K) >= 3 * K + D, "the triangle area holds the parts of t and the row");
        float *p1 = tri, *p2 = tri + K, *zeros = tri + 2 * K, *rbuf = tri + 3 * K;
#pragma unroll
        for (int e0 = 0; e0 < K; e0 += 64) {
            const int e = e0 + lane;
            if (e < K) {
                float x1, x2;
                t_parts(tbuf[e], x1, x2);
                p1[e] = x1;
                p2[e] = x2;
                zeros[e] = 0.f;
            }
        }
        const SelOperands sel = make_sel(lane);
        wave_sync();
        const float *mine = (a == 0 ? tbuf : (a == 1 ? p1 : (a == 2 ? p2 : zeros))) + 4 * q;
        bf16x8 top[(KT + 1) / 2];
#pragma unroll
        for (int P = 0; P < (KT + 1) / 2; ++P) top[P] = t_operand(mine + 32 * P, 2 * P + 1 < KT);
        constexpr int NP = D / 32;
        floatx4 out[2 * NP];
#pragma unroll
        for (int x = 0; x < 2 * NP; ++x) out[x] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (ZB)
            zt_times_t<KT, NP>([&](int t, int j) { return __builtin_bit_cast(bf16x8, zop[t].v[j]); }, top, sel, out);
        float *dump = aux + TRI_AUX_DUMP<K> + lane;  // the solver's per-lane dump slots
#pragma unroll
        for (int x = 0; x < 2 * NP; ++x)
            *(q == 0 ? rbuf + column_of_result(x >> 1, x & 1, a) : dump) = out[x][0] + out[x][1] + out[x][2];
        wave_sync();
        if constexpr (D >= 128) *(float2 *)(R + u * ldr + 2 * lane) = *(const float2 *)(rbuf + 2 * lane);
        else R[u * ldr + lane] = rbuf[lane];
    } else {
        // 16 bytes of an entry per lane, GatherCols<D>::EPI entries per instruction, four entries per lane and round, the loads of
        // four rounds under way together (10M pages, d = 128, KT = 4 .. 8: a round at a time 3.71, 2.63, 1.89, 1.65, 1.00 ms; so 3.63,
        // 2.52, 1.75, 1.30, 0.80, the last two with more tiles resident too, see wide_tiles).  Not where conjugate gradients bring rows of up
        // to 48 entries: 60 000 rows of 25 / of 33 to 48 281 / 402 us a round at a time, 296 / 417 with four.
        using GC = GatherCols<D>;
        constexpr int ROUND = 4 * GC::EPI, AHEAD = CG && KT == 3 ? 1 : (K / ROUND < 4 ? K / ROUND : 4);
        const int mine = 4 * (lane / GC::LPR);
        const float *col = (const float *)Z + 4 * (lane % GC::LPR);
        floatx4 rv = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int e0 = 0; e0 < k; e0 += AHEAD * ROUND) {  // padded entries have t = 0 and the id of the row's first entry
            // ids and t with 16-byte LDS reads, before the first load is issued
            int4 id4[AHEAD];
            float4 t4[AHEAD];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const int e = K % (AHEAD * ROUND) == 0 || e0 + u * ROUND < K ? e0 + u * ROUND : 0;  // beyond the last place: not used
                id4[u] = *(const int4 *)(ids + e + mine);
                t4[u] = *(const float4 *)(tbuf + e + mine);
            }
            floatx4 zz[AHEAD][4];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
                if (u == 0 || e0 + u * ROUND < k) {  // uniform
                    const int id[4] = {id4[u].x, id4[u].y, id4[u].z, id4[u].w};
#pragma unroll
                    for (int x = 0; x < 4; ++x) zz[u][x] = *(const floatx4 *)(col + (int64_t)id[x] * D);
                }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
                if (u == 0 || e0 + u * ROUND < k) {
                    const float te[4] = {t4[u].x, t4[u].y, t4[u].z, t4[u].w};
#pragma unroll
                    for (int x = 0; x < 4; ++x)
#pragma unroll
                        for (int c = 0; c < 4; ++c) rv[c] += te[x] * zz[u][x][c];
                }
        }
        rv = swap_add32(rv, rv);
        if constexpr (D == 64) rv = swap_add16(rv, rv);
        if (lane < GC::LPR) *(floatx4 *)(R + u * ldr + 4 * lane) = rv;
    }
}

}  // namespace als
