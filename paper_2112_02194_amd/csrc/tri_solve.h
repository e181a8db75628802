// One wavefront solves a symmetric positive definite K x K system (K <= 128, a multiple of 16) whose
// lower triangle sits in LDS, row r starting at tri_row<K>(r).  Rows are padded to multiples of sixteen floats:
// a row at or below a panel of 16 columns then holds all 16 of them inside its own storage (beyond its
// diagonal: padding, never used), so a panel is read and written back with 16-byte accesses and no
// per-element test.
//
// Blocked elimination S = M P M^T (M unit lower triangular, P the pivots) with panels of 16 columns.
// Lane i owns rows i and 64+i.  Per panel:
//   1. every lane reads the panel's 16 entries of its rows into registers and the 16 columns are
//      eliminated there: pivot, column entries and right-hand-side entry of a step are read from the
//      owning lanes as wavefront-uniform values (no memory traffic, no synchronisation); the reciprocal
//      pivot of the next step is prepared right after that column's first update; u = M^{-1} y rides
//      along;
//   2. the eliminated entries S' go back to LDS and the trailing matrix is updated there on the matrix
//      cores: for 16 x 16 tiles (ti, tj <= ti) below the panel, S[ti][tj] -= (S' P^{-1})[ti] S'[tj]^T.
//      Lane (a, q) = (lane % 16, lane / 16) of v_mfma_f32_16x16x4f32 supplies A[a][q] and B[q][a] and
//      holds C[4q+v][a]; MFMA e of a tile contracts the panel columns 4q + e, so that every lane fetches
//      its operands of the four MFMAs with one 16-byte read; the tile is computed transposed (A from the
//      column tile's rows, B from the row tile's), so that C[4q+v][a] is row a, columns 4q+v of the tile.
// Then back-substitution t_c = (u_c - sum_{R>c} S'[R][c] t_R) / pivot_c along the rows of the factor in
// LDS, eight rows fetched ahead of the dependent chain; the value just found is read from its lane.
// Panels and steps at or beyond k are skipped: the caller guarantees that rows >= k are identity rows
// with zero right-hand side.  y0 / y1: right-hand-side entries of rows lane / 64+lane.  On exit
// tbuf[0..K) holds the solution.  A non-positive pivot sets bit 0 of *err_flag.
#pragma once

#include "dual_common.h"

namespace als {

// First float of row r in the padded triangle; tri_row<K>(K) is the size of the whole triangle.  Beyond 64 rows every row
// starts four floats further on: with row lengths of 16 to 128 floats alone, sixteen lanes that read 16 bytes each
// from sixteen rows meet in one to four groups of four banks, with the shift in sixteen different ones (a power-law
// epoch of 50M rows, bf16, d = 128: 259 -> 253 ms).  Up to 64 rows the shift costs more resident workgroups than it gains.
template <int K> __host__ __device__ constexpr int tri_row(int r) {
    return 16 * (r / 16 + 1) * (8 * (r / 16) + r % 16) + (K > 64 ? 4 * r : 0);
}

// reciprocal pivots, then the callers' 64 per-lane dump slots
template <int K> constexpr int TRI_AUX_DUMP = K > 64 ? 128 : 64;
template <int K> constexpr int TRI_AUX_FLOATS = TRI_AUX_DUMP<K> + 64;

__device__ __forceinline__ float lane_value(float v, int src_lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src_lane));
}

// v with the wavefront-uniform value `uniform` put into lane DST (one instruction; the lane is a constant, so
// the instruction's wait states for a lane select computed just before do not apply)
template <int DST> __device__ __forceinline__ float lane_set(float v, float uniform) {
    asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(uniform), "n"(DST));
    return v;
}

// Back-substitution of the eliminated system by one wavefront: y0 / y1 hold u = M^-1 y and rp0 / rp1 the reciprocal
// pivots of rows lane / 64+lane.
template <int K>
__device__ __forceinline__ void tri_back(const float *tri, float *tbuf, float y0, float y1, float rp0, float rp1, int k) {
    const int lane = opaque_tid() & 63;
    // Eight rows of the factor fetched ahead of the dependent chain.  Every lane reads
    // row R at its own column: lanes at or beyond R have their unknown already and go on computing on
    // whatever lies there (the row's padding, later rows, at most the first 127 floats after the triangle - 63 for
    // K <= 64 -, which every caller's LDS layout has).  Groups of rows at or beyond k hold t = 0.
    float t0 = 0.f, t1v = 0.f;
    static_for<0, K / 8>([&](auto gg) {
        constexpr int Rt = K - 1 - 8 * decltype(gg)::value;  // the group's last row; rows Rt-7 .. Rt
        if (Rt - 7 < k) {
            float fa[8], fb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int Rr = Rt - i;
                const float *row = tri + tri_row<K>(Rr);
                fa[i] = row[lane];
                if (Rr >= 64) fb[i] = row[64 + lane];
            }
            static_for<0, 8>([&](auto ii) {
                constexpr int i = decltype(ii)::value, Rr = Rt - i;
                if constexpr (Rr >= 64) {
                    const float tR = lane_value(y1 * rp1, Rr - 64);
                    t1v = lane_set<Rr - 64>(t1v, tR);
                    y1 -= fb[i] * tR;
                    y0 -= fa[i] * tR;
                } else {
                    const float tR = lane_value(y0 * rp0, Rr);
                    t0 = lane_set<Rr>(t0, tR);
                    y0 -= fa[i] * tR;
                }
            });
        }
    });
    if (lane < K) tbuf[lane] = t0;
    if (K > 64 && 64 + lane < K) tbuf[64 + lane] = t1v;
    wave_sync();
}

template <int K>
__device__ __forceinline__ void tri_solve(float *tri, float *aux /* [TRI_AUX_FLOATS<K>] */, float *tbuf /* [K] */, float y0,
                                          float y1, int k, int32_t *err_flag) {
    static_assert(K % 16 == 0 && K >= 16 && K <= 128, "unsupported system size");
    constexpr bool TWO = K > 64;
    constexpr int NT = K / 16;
    const int lane = opaque_tid() & 63;
    const int ra = lane, rb = 64 + lane;
    const bool hasa = ra < K, hasb = TWO && rb < K;
    const int a = lane & 15, q = lane >> 4;
    float *rpbuf = aux;
    float *rowa = tri + tri_row<K>(hasa ? ra : 0), *rowb = tri + tri_row<K>(hasb ? rb : 0);
    float rp0 = 1.f, rp1 = 1.f;
    static_for<0, NT>([&](auto pp) {
        constexpr int p = decltype(pp)::value;
        constexpr int P0 = 16 * p;
        constexpr bool OB = P0 >= 64;  // the panel's pivot rows belong to the second set of rows
        if (P0 < k) {
            // Every lane reads 16 floats at the panel's columns of its rows.  What is not an entry of the matrix
            // there (beyond a row's diagonal; a row above the panel; a lane without a row) is never used: the
            // multipliers below are taken only for rows under the pivot, lane reads only go to lanes whose entry
            // exists, and only rows at or below the panel are written back.
            float xa[16], xb[16];
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) {
                float4 va = make_float4(0.f, 0.f, 0.f, 0.f), vb = va;
                if constexpr (!OB) va = *(const float4 *)(rowa + P0 + 4 * c4);
                if constexpr (TWO) vb = *(const float4 *)(rowb + P0 + 4 * c4);
                xa[4 * c4] = va.x; xa[4 * c4 + 1] = va.y; xa[4 * c4 + 2] = va.z; xa[4 * c4 + 3] = va.w;
                xb[4 * c4] = vb.x; xb[4 * c4 + 1] = vb.y; xb[4 * c4 + 2] = vb.z; xb[4 * c4 + 3] = vb.w;
            }
            // reciprocal pivot and right-hand-side entry of a step are prepared during the step before
            // (right after its first update), off the critical path
            float rp, uc;
            auto prepare = [&](auto cc) {
                constexpr int c = decltype(cc)::value;
                constexpr int ol = (P0 + c) & 63;
                const float pivot = lane_value(OB ? xb[c] : xa[c], ol);
                rp = __builtin_amdgcn_rcpf(pivot);
                rp = rp * (2.f - pivot * rp);  // one Newton step on the hardware reciprocal
                if constexpr (OB) rp1 = lane == ol ? rp : rp1;
                else rp0 = lane == ol ? rp : rp0;
            };
            prepare(std::integral_constant<int, 0>{});
            static_for<0, 16>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                constexpr int col = P0 + c, ol = col & 63;
                if (col < k) {
                    const float own = OB ? xb[c] : xa[c];
                    float cv[16];
#pragma unroll
                    for (int j = c + 1; j < 16; ++j) cv[j] = lane_value(own, (P0 + j) & 63);
                    uc = lane_value(OB ? y1 : y0, ol);
                    float fa = 0.f, fb = 0.f;
                    if constexpr (!OB) {
                        fa = ra > col ? xa[c] * rp : 0.f;
                        y0 -= fa * uc;
                    }
                    if constexpr (TWO) {
                        fb = (!OB || rb > col) ? xb[c] * rp : 0.f;
                        y1 -= fb * uc;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (c < 15) {
                        if constexpr (!OB) xa[c + 1] -= fa * cv[c + 1];
                        if constexpr (TWO) xb[c + 1] -= fb * cv[c + 1];
                        prepare(std::integral_constant<int, c + 1>{});
#pragma unroll
                        for (int j = c + 2; j < 16; ++j) {
                            if constexpr (!OB) xa[j] -= fa * cv[j];
                            if constexpr (TWO) xb[j] -= fb * cv[j];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            if constexpr (!OB) {
                if (hasa && ra >= P0) {
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4)
                        *(float4 *)(rowa + P0 + 4 * c4) = make_float4(xa[4 * c4], xa[4 * c4 + 1], xa[4 * c4 + 2], xa[4 * c4 + 3]);
                }
            }
            if constexpr (TWO) {
                if (hasb && rb >= P0) {
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4)
                        *(float4 *)(rowb + P0 + 4 * c4) = make_float4(xb[4 * c4], xb[4 * c4 + 1], xb[4 * c4 + 2], xb[4 * c4 + 3]);
                }
            }
            rpbuf[lane] = rp0;
            if constexpr (TWO) rpbuf[64 + lane] = rp1;
            wave_sync();
            if constexpr (p + 1 < NT) {
                constexpr int T = NT - p - 1;
                const float4 rpv = *(const float4 *)(rpbuf + P0 + 4 * q);
                float4 z[T];
#pragma unroll
                for (int t = 0; t < T; ++t) z[t] = *(const float4 *)(tri + tri_row<K>(16 * (p + 1 + t) + a) + P0 + 4 * q);
                static_for<0, T>([&](auto tii) {
                    constexpr int ti = decltype(tii)::value;
                    const float4 za = make_float4(-z[ti].x * rpv.x, -z[ti].y * rpv.y, -z[ti].z * rpv.z, -z[ti].w * rpv.w);
                    // all tiles of the tile row are fetched before the first is stored back.  The operands are taken
                    // in the order that leaves a lane with four consecutive columns of ONE row of the tile (row
                    // 16 (p+1+ti) + a, columns 16 (p+1+tj) + 4q ..): one 16-byte access each way; in a diagonal tile
                    // the columns beyond the diagonal belong to the row's padding
                    floatx4 acc[ti + 1];
                    float4 *cell[ti + 1];
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) {
                        cell[tj] = (float4 *)(tri + tri_row<K>(16 * (p + 1 + ti) + a) + 16 * (p + 1 + tj) + 4 * q);
                        const float4 c4 = *cell[tj];
                        acc[tj] = floatx4{c4.x, c4.y, c4.z, c4.w};
                    }
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) acc[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[tj].x, za.x, acc[tj], 0, 0, 0);
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) acc[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[tj].y, za.y, acc[tj], 0, 0, 0);
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) acc[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[tj].z, za.z, acc[tj], 0, 0, 0);
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) acc[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[tj].w, za.w, acc[tj], 0, 0, 0);
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) *cell[tj] = make_float4(acc[tj][0], acc[tj][1], acc[tj][2], acc[tj][3]);
                });
                wave_sync();
            }
        }
    });
    // A pivot that is not positive shows in its reciprocal, which the owning lane has kept: negative stays
    // negative, zero and NaN come out of the Newton step as NaN.
    if (__any(!(rp0 > 0.f) || !(rp1 > 0.f)) && lane == 0) atomicOr(err_flag, 1);

    tri_back<K>(tri, tbuf, y0, y1, rp0, rp1, k);
}
// Sum over the four rows of 16 lanes, in every lane.
__device__ __forceinline__ float sum_lane_rows(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float w = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(w), __float_as_uint(w), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// Sum over the 16 lanes of this lane's row, in every lane.
__device__ __forceinline__ float sum_lane_row(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true));  // row_ror:8
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, true));
    return v;
}

// The same for one or two panels, S = M P M^T by blocks.  Lane (i, q) = (lane % 16, lane / 16).  Per panel p:
//   1. the 16 x 16 diagonal block is eliminated in registers, in place: lane (i, q) holds the entries (i, 4 q + s), and a
//      column that is done makes room for the same column of N = M_pp^{-1}.  A step takes four multiply-adds (the pivot row
//      comes as a DPP modifier) instead of up to fifteen with a lane read each, the pivot from its lane, the pivot column by
//      lane swaps.
//   2. u_p = N y_p.
//   3. the tile below becomes W = A N^T on the matrix cores: v_mfma_f32_16x16x4f32 takes A[a][q] and B[q][a] from lane
//      (a, q) and leaves C[4q+v][a]; instruction e contracts the columns 4q + e, so N as it stands in the registers is one
//      operand, 16 bytes of a tile row the other, and the result (computed transposed) is row a, columns 4q .. of W.
//   4. the tile after it is updated the same way, A -= W P^{-1} W^T, and y -= W P^{-1} u_p.
// Then, from the last panel to the first, t_p = N^T P^{-1} (u_p - W^T t).
// What bounds it: the chain of the steps, and with many rows per SIMD their instructions.  Epoch of 50k x 30k with labels (d = 32,
// half of the rows longer than 32): the kernel 177 -> 167 us, the epoch 335 -> 325 us.  For 48 <= K <= 128 the form above is
// the better one: a step's chain is longer here (10M pages, d = 128, fp32: 0 to 1 % slower, 50M rows bf16: 1 %).
template <int K>
__device__ __forceinline__ void block_solve(float *tri, float *aux /* [TRI_AUX_FLOATS<K>] */, float *tbuf /* [K] */, float y0,
                                            int k, int32_t *err_flag) {
    static_assert(K == 16 || K == 32, "unsupported system size");
    constexpr int NT = K / 16;
    const int lane = opaque_tid() & 63, a = lane & 15, q = lane >> 4;
    bool bad = false;
    if (lane < K) tbuf[lane] = y0;  // y, then u, then t
    wave_sync();
    static_for<0, NT>([&](auto pp) {
        constexpr int p = decltype(pp)::value, P0 = 16 * p, T = NT - p - 1;
        if (P0 < k) {
            float x[4], mine = 1.f;
            floatx4 z[T > 0 ? T : 1];
#pragma unroll
            for (int s = 0; s < 4; ++s) {  // the lower triangle is what callers fill
                const int c = 4 * q + s;
                x[s] = c <= a ? tri[tri_row<K>(P0 + a) + P0 + c] : tri[tri_row<K>(P0 + c) + P0 + a];
            }
            const floatx4 yv = *(const floatx4 *)(tbuf + P0 + 4 * q);
            dpp_settle(x);
            static_for<0, 16>([&](auto cc) {
                constexpr int c = decltype(cc)::value, sc = c & 3, qc = c >> 2;
                if (P0 + c < k) {
                    const float pivot = lane_value(x[sc], 16 * qc + c);
                    float rp = __builtin_amdgcn_rcpf(pivot);
                    rp = rp * (2.f - pivot * rp);  // one Newton step on the hardware reciprocal
                    mine = a == c ? rp : mine;
                    const float col = from_lane_row<qc>(x[sc]);
                    const float f = a > c ? col * rp : 0.f;
                    const float done = a == c ? 1.f : -f;  // this row's entry of N in column c
#pragma unroll
                    for (int s = 0; s < 4; ++s) fmac_bcast16_neg_self<c>(x[s], f);
                    x[sc] = q == qc ? done : x[sc];
                    dpp_settle(x);
                }
            });
            bad |= !(mine > 0.f);  // negative stays negative, zero and NaN come out of the Newton step as NaN
            const float u = sum_lane_rows(x[0] * yv[0] + x[1] * yv[1] + x[2] * yv[2] + x[3] * yv[3]);
            tbuf[P0 + a] = u;  // four lanes, the same value
            aux[P0 + a] = mine;
            *(floatx4 *)(tri + tri_row<K>(P0 + a) + P0 + 4 * q) = floatx4{x[0], x[1], x[2], x[3]};
            wave_sync();
            if constexpr (T > 0) {
                const floatx4 rpv = *(const floatx4 *)(aux + P0 + 4 * q), uv = *(const floatx4 *)(tbuf + P0 + 4 * q);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    floatx4 *cell = (floatx4 *)(tri + tri_row<K>(16 * (p + 1 + t) + a) + P0 + 4 * q);
                    const floatx4 c4 = *cell;
                    floatx4 w = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) w = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], c4[e], w, 0, 0, 0);
                    z[t] = w;
                    *cell = w;
                }
                static_for<0, T>([&](auto tii) {
                    constexpr int ti = decltype(tii)::value;
                    floatx4 za;
#pragma unroll
                    for (int e = 0; e < 4; ++e) za[e] = -z[ti][e] * rpv[e];
                    const float d = sum_lane_rows(za[0] * uv[0] + za[1] * uv[1] + za[2] * uv[2] + za[3] * uv[3]);
                    tbuf[16 * (p + 1 + ti) + a] += d;
                    // all tiles of the tile row are fetched before the first is stored back; in a diagonal tile the columns
                    // beyond the diagonal belong to the row's padding
                    floatx4 acc[ti + 1];
                    floatx4 *cell[ti + 1];
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) {
                        cell[tj] = (floatx4 *)(tri + tri_row<K>(16 * (p + 1 + ti) + a) + 16 * (p + 1 + tj) + 4 * q);
                        acc[tj] = *cell[tj];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int tj = 0; tj <= ti; ++tj) acc[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[tj][e], za[e], acc[tj], 0, 0, 0);
#pragma unroll
                    for (int tj = 0; tj <= ti; ++tj) *cell[tj] = acc[tj];
                });
                wave_sync();
            }
        }
    });
    if (__any(bad) && lane == 0) atomicOr(err_flag, 1);
    static_for<0, NT>([&](auto pp) {
        constexpr int p = NT - 1 - decltype(pp)::value, P0 = 16 * p, T = NT - p - 1;
        if (P0 < k) {
            floatx4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const floatx4 w = *(const floatx4 *)(tri + tri_row<K>(16 * (p + 1 + t) + a) + P0 + 4 * q);
                const float ti = tbuf[16 * (p + 1 + t) + a];
#pragma unroll
                for (int s = 0; s < 4; ++s) s4[s] += w[s] * ti;
            }
            const floatx4 n4 = *(const floatx4 *)(tri + tri_row<K>(P0 + a) + P0 + 4 * q);
            const floatx4 rpv = *(const floatx4 *)(aux + P0 + 4 * q), uv = *(const floatx4 *)(tbuf + P0 + 4 * q);
            floatx4 v4;
#pragma unroll
            for (int s = 0; s < 4; ++s) v4[s] = rpv[s] * (uv[s] - (T > 0 ? sum_lane_row(s4[s]) : 0.f));
            wave_sync();
            *(floatx4 *)(tbuf + P0 + 4 * q) = v4;  // sixteen lanes, the same values
            wave_sync();
            const float va = tbuf[P0 + a];
            floatx4 t4;
#pragma unroll
            for (int s = 0; s < 4; ++s) t4[s] = sum_lane_row(n4[s] * va);
            wave_sync();
            *(floatx4 *)(tbuf + P0 + 4 * q) = t4;
            wave_sync();
        }
    });
}

// The elimination of tri_solve by a workgroup of four wavefronts, for systems too few per compute unit to hide one wavefront's
// chain (K = 128: a workgroup's triangle takes a quarter of the LDS).  Every wavefront that works on a panel eliminates the
// panel's 16 pivot rows for itself (lanes 0 .. 15) and 48 of the rows below in its other lanes - the steps cost what
// they cost with 16 rows, nothing is exchanged between wavefronts, and the numbers are those of tri_solve -, and the tiles
// of the trailing update are dealt out to all four.  rhs[K] in LDS: y on entry, u = M^-1 y on exit; aux[0..K): reciprocal
// pivots.  Called by all 256 threads behind a barrier; wavefront 0 returns last and may read what it and the others have
// left in LDS, the others must not touch the LDS again before the next barrier.
// With one wavefront the solve took 57 000 of a row's 131 000 clocks in the 50M-row power-law epoch (d = 128, bf16).
template <int K>
__device__ __forceinline__ void team_tri_eliminate(float *tri, float *aux, float *rhs, int wave_s, int32_t *err_flag) {
    constexpr int NT = K / 16;
    const int lane = opaque_tid() & 63, a = lane & 15, q = lane >> 4;
    bool bad = false;
    static_for<0, NT>([&](auto pp) {
        constexpr int p = decltype(pp)::value, P0 = 16 * p, BELOW = K - P0 - 16, W = BELOW > 0 ? (BELOW + 47) / 48 : 1;
        float x[16], y = 0.f;
        const int row = lane < 16 ? P0 + lane : P0 + 48 * wave_s + lane;
        const bool has = row < K;
        float *cells = tri + tri_row<K>(has ? row : P0) + P0;
        if (wave_s < W) {  // scalar branch
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) {
                const float4 v = *(const float4 *)(cells + 4 * c4);
                x[4 * c4] = v.x; x[4 * c4 + 1] = v.y; x[4 * c4 + 2] = v.z; x[4 * c4 + 3] = v.w;
            }
            y = rhs[has ? row : P0];
            float rp, mine = 1.f;
            auto prepare = [&](auto cc) {
                constexpr int c = decltype(cc)::value;
                const float pivot = lane_value(x[c], c);
                rp = __builtin_amdgcn_rcpf(pivot);
                rp = rp * (2.f - pivot * rp);  // one Newton step on the hardware reciprocal
                mine = lane == c ? rp : mine;
            };
            prepare(std::integral_constant<int, 0>{});
            static_for<0, 16>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                float cv[16];
#pragma unroll
                for (int j = c + 1; j < 16; ++j) cv[j] = lane_value(x[c], j);
                const float uc = lane_value(y, c);
                const float f = lane > c ? x[c] * rp : 0.f;
                y -= f * uc;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (c < 15) {
                    x[c + 1] -= f * cv[c + 1];
                    prepare(std::integral_constant<int, c + 1>{});
#pragma unroll
                    for (int j = c + 2; j < 16; ++j) x[j] -= f * cv[j];
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if (lane >= 16 && has) {
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4) *(float4 *)(cells + 4 * c4) = make_float4(x[4 * c4], x[4 * c4 + 1], x[4 * c4 + 2], x[4 * c4 + 3]);
                rhs[row] = y;
            }
            if (wave_s == 0 && lane < 16) aux[P0 + lane] = mine;
            bad = bad || !(mine > 0.f);
        }
        if constexpr (p + 1 < NT) __syncthreads();
        // the pivot rows go back only now that no wavefront can still be reading them
        if (wave_s == 0 && lane < 16) {
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) *(float4 *)(cells + 4 * c4) = make_float4(x[4 * c4], x[4 * c4 + 1], x[4 * c4 + 2], x[4 * c4 + 3]);
            rhs[row] = y;
        }
        if constexpr (p + 1 < NT) {
            constexpr int T = NT - p - 1, TILES = T * (T + 1) / 2, PER = (TILES + 3) / 4, GRP = 4;
            const float4 rpv = *(const float4 *)(aux + P0 + 4 * q);
            auto block_row = [&](int b) { return tri + (128 * b * (b + 1) + (K > 64 ? 64 * b : 0)) + (16 * (b + 1) + (K > 64 ? 4 : 0)) * a; };
            static_for<0, (PER + GRP - 1) / GRP>([&](auto gg) {
                constexpr int g0 = decltype(gg)::value * GRP, N = PER - g0 < GRP ? PER - g0 : GRP;
                float4 zj[N], za[N], *cell[N];
                floatx4 acc[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const int t = wave_s + 4 * (g0 + u) < TILES ? wave_s + 4 * (g0 + u) : 0;  // tile (ti, tj <= ti) in row order
                    const int ti = (t >= 1) + (t >= 3) + (t >= 6) + (t >= 10) + (t >= 15) + (t >= 21), tj = t - ti * (ti + 1) / 2;
                    const float *ri = block_row(p + 1 + ti);
                    const float4 zi = *(const float4 *)(ri + P0 + 4 * q);
                    zj[u] = *(const float4 *)(block_row(p + 1 + tj) + P0 + 4 * q);
                    cell[u] = (float4 *)(ri + 16 * (p + 1 + tj) + 4 * q);
                    const float4 c4 = *cell[u];
                    acc[u] = floatx4{c4.x, c4.y, c4.z, c4.w};
                    za[u] = make_float4(-zi.x * rpv.x, -zi.y * rpv.y, -zi.z * rpv.z, -zi.w * rpv.w);
                }
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(zj[u].x, za[u].x, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(zj[u].y, za[u].y, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(zj[u].z, za[u].z, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(zj[u].w, za[u].w, acc[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < N; ++u)
                    if (wave_s + 4 * (g0 + u) < TILES) *cell[u] = make_float4(acc[u][0], acc[u][1], acc[u][2], acc[u][3]);
            });
            __syncthreads();
        }
    });
    wave_sync();
    // a pivot that is not positive shows in its reciprocal (see tri_solve)
    if (wave_s == 0 && __any(bad && lane < 16) && lane == 0) atomicOr(err_flag, 1);
}

}  // namespace als
