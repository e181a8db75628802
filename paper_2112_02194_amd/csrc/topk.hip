// Exact top-k retrieval by inner product: for every query row, the k rows of an item table with the largest
// <query, item>.  The paper names top-K retrieval as the step after training (Section 4.6) and evaluates with
// Recall@20 / Recall@50 on test rows whose embedding is folded in with Eq. 4 from part of their links
// (Section 5); the folded-in rows come from als_solve_rows, this file supplies the retrieval.
//
// Almost no item is among a query's best, so the full-accuracy score of an item is computed only where a cheap bound
// cannot rule the item out:
//
// bound kernel   scores all (query, item) pairs on the bf16 matrix cores (fp32 entries rounded to bf16, bf16 entries as
//                they are) and keeps, per query and chunk of C items, nothing but the largest one; per chunk also the
//                largest item norm.  By Cauchy-Schwarz a bf16 score is within eps |query| |item| of the exact one
//                (`margin`), so the chunk's best exact score lies within margin of the stored maximum.
// select kernel  one workgroup per query.  k chunks whose best is at least some value hold k different items that
//                are at least that good, so the k-th largest lower bound is a bar that the k-th best item clears
//                (chunks with excluded items do not count for the bar).  The chunks whose upper bound reaches the
//                bar, little more than k of them, are scored again in full (score_tile), the survivors checked
//                against the exclusion list, sorted, and the best k written.
// Where many chunks reach the bar (nearly parallel rows, ties, a query without a bound) rescoring would walk the table once
// per query and share nothing.  Such queries are left to
//
// scan kernel    a wavefront owns 16 of them (their operand registers stay loaded) and walks the item tiles of its slice
//                of the table, 16 items at a time, with score_tile.  A score at least as large as the query's current
//                k-th best is appended to the query's candidate buffer in LDS (after a look at the query's exclusion
//                list); a buffer that fills up is sorted by the wavefront and cut back to its best k, which also raises
//                the bar.  The four wavefronts of a workgroup walk the same tiles for 64 different queries, so a tile
//                comes from HBM once per 64 queries.  Each slice leaves its best k per query in a workspace.
// merge kernel   one wavefront per query sorts the slices' candidates and writes the best k.
//
// Order everywhere: descending score, equal scores by ascending item id, so the result is unique.  What cannot be
// bounded (entries that are infinite, NaN or so large that a product may overflow) has an infinite margin: it never
// sets the bar and is always scored exactly.
#include <cmath>

#include "dual_common.h"
#include "row_piece.h"
#include "topk_batch.h"

namespace als {

constexpr int TOPK_SEG = 32;      // items of one matrix-core tile; a chunk is made of such segments
constexpr int TOPK_CAND = 1024;   // candidate slots of the select kernel
constexpr int TOPK_LIST = 2048;   // chunks listed for rescoring at a time
constexpr int TOPK_ROUND = 6;     // segments per wavefront between two looks at the candidate count
constexpr int SCAN_CAP = 128;       // scan: candidate slots per query in LDS
constexpr int SCAN_MERGE = 1024;    // candidates the merge sorts per query (slices * padded k)
constexpr int SCAN_QPW = 16, SCAN_WAVES = 4;
constexpr int SCAN_TILES = 2;       // tiles of 16 items a wavefront scores per round
constexpr int TOPK_MAX_CHUNKS = 1 << 18;  // the select kernel's chunk bitmap takes 32 KB of LDS
static_assert(4 * TOPK_ROUND * TOPK_SEG + ALS_TOPK_MAX_K <= TOPK_CAND, "a round must fit behind the kept candidates");
static_assert(ALS_TOPK_MAX_K <= 256, "the bar is the k-th largest of 256 thread maxima");

// Items are grouped in units of four chunks: segment j of a unit (32 consecutive items) belongs to chunk j % 4 of
// the unit, so that a workgroup finishes four chunks together, whether its wavefronts share the segments or the queries.
struct ChunkMap {
    int lc;       // log2 of the items per chunk
    int nchunks;  // four per unit
    __host__ __device__ int64_t unit_items() const { return (int64_t)4 << lc; }
    __device__ int64_t first(int c) const { return ((int64_t)(c >> 2) << (lc + 2)) + TOPK_SEG * (c & 3); }
    __device__ int64_t segment(int c, int r) const { return first(c) + (int64_t)r * 4 * TOPK_SEG; }
    __device__ int of_item(int64_t i) const { return (int)(i >> (lc + 2)) * 4 + (int)((i / TOPK_SEG) & 3); }
    __device__ bool complete(int c, int64_t n) const { return segment(c, (1 << (lc - 5)) - 1) + TOPK_SEG <= n; }
};
// maxima[(c / 16 * nq + query) * 16 + c % 16]: a wavefront's store covers neighbouring queries, a query's reads 64 bytes
__device__ __forceinline__ int64_t maxima_at(int c, int64_t q, int64_t nq) { return ((int64_t)(c >> 4) * nq + q) * 16 + (c & 15); }

// The piece as a matrix-core operand: fp32 entries rounded to nearest.
template <bool BF16> __device__ __forceinline__ bf16x8 piece_bf16(const Piece<BF16> &p) {
    if constexpr (BF16) {
        return __builtin_bit_cast(bf16x8, p.v[0]);
    } else {
        typedef float floatx8 __attribute__((ext_vector_type(8)));
        const floatx8 f = {p.v[0].x, p.v[0].y, p.v[0].z, p.v[0].w, p.v[1].x, p.v[1].y, p.v[1].z, p.v[1].w};
        return __builtin_convertvector(f, bf16x8);
    }
}

// Upper bound of a row's 2-norm from its sum of squares and largest magnitude (the squares of very small entries
// underflow; NaN and infinity stay: fmaxf drops a NaN entry from amax, the sum keeps it).
__device__ __forceinline__ float norm_bound(float sumsq, float amax, int d) {
    return !(sumsq < 1e-24f) || !(amax < 1.f) ? sqrtf(sumsq) * 1.00001f : amax * sqrtf((float)d);
}
// |bf16 score - computed fp32 score| <= margin: both operands rounded to bf16 (2^-8 each) for fp32 tables, exact
// products otherwise; d 2^-21 covers the fp32 sums of both sides however they are ordered or rounded, the last term
// entries and products below the normal range.
template <int D, bool BF16> __device__ __forceinline__ float margin(float qn, float hn) {
    constexpr float eps = (BF16 ? 0.f : 0.0079f) + D * 4.8e-7f;
    const float p = qn * hn;
    if (!(p < 1e37f)) return INFINITY;
    return qn == 0.f || hn == 0.f ? 0.f : eps * p + 4e-36f * (1.f + qn + hn);
}

// What bounds it: the matrix cores and the barriers between stages once a few hundred queries share an item (4096 queries x
// 10M bf16 items, d = 128: about 8.5 ms, 1.2 PFLOP/s), the item table's read below that.  A workgroup stages a stretch of items in LDS once (coalesced, converted, its rows
// padded by 16 bytes against bank conflicts) and its wavefronts multiply it with queries kept in registers: WI = 1
// gives every wavefront its own QT * 32 queries and all items, WI = 4 the same QT * 32 queries and a quarter of the items.
template <int D, int WI> constexpr int topk_stage_items() { return WI == 4 || D == 16 ? 128 : 64; }
template <int QT, int WI> constexpr int topk_group_queries() { return 32 * QT * (4 / WI); }

template <int D, bool BF16, int QT, int WI>
__global__ __launch_bounds__(256, 2) void topk_bound_kernel(const void *__restrict__ Q, int64_t ldq, int64_t nq,
                                                            const void *__restrict__ H, int64_t ldh, int64_t n,
                                                            ChunkMap map, unsigned qgroups, int64_t units_per_group,
                                                            float *__restrict__ maxima, float *__restrict__ norms,
                                                            int32_t *__restrict__ deferred) {
    constexpr int S = topk_stage_items<D, WI>(), PITCH = 2 * D + 16, PPR = D / 8;
    constexpr int NP = S * PPR / 256, KS = D / 16, SUB = WI == 1 ? S / TOPK_SEG : 1, NM = WI == 1 ? 4 : 1;
    static_assert(NP >= 1 && S * PPR % 256 == 0, "every thread stages the same number of pieces");
    __shared__ __align__(16) char lds[2][S * PITCH];
    __shared__ unsigned nmax[2][4];  // largest norm of a chunk (as bits: they order like the values, NaN last), by unit parity
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, a = lane & 31, h = lane >> 5;
    if (blockIdx.x == 0 && tid == 0) deferred[0] = 0;
    // Consecutive workgroups go to different XCDs: those that read the same items for other queries sit 8 apart, so that
    // they meet in one L2.
    const unsigned slot = blockIdx.x >> 3;
    const unsigned qg = slot % qgroups;
    const int64_t split = (int64_t)(slot / qgroups) * 8 + (blockIdx.x & 7);
    const int64_t units = map.nchunks / 4;
    const int64_t u0 = split * units_per_group, u1 = u0 + units_per_group < units ? u0 + units_per_group : units;
    if (u0 >= u1) return;
    const int spu = (int)(map.unit_items() / S);  // stages per unit; even for S = 64
    const int64_t item_base = u0 * map.unit_items(), stages = (u1 - u0) * spu;
    const bool with_norms = qg == 0;

    int64_t query[QT];
    bf16x8 bq[QT][KS];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        query[t] = (int64_t)qg * topk_group_queries<QT, WI>() + (WI == 1 ? wave * 32 * QT : 0) + 32 * t + a;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            Piece<BF16> p = piece_zero<BF16>();
            if (query[t] < nq) p = piece_load<BF16>(Q, query[t] * ldq + (2 * s + h) * 8);
            bq[t][s] = piece_bf16<BF16>(p);
        }
    }

    Piece<BF16> raw[NP];
    auto fetch = [&](int64_t stage) {
        const int64_t t0 = item_base + stage * S;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int p = i * 256 + tid;
            const int64_t item = t0 + p / PPR;
            raw[i] = piece_zero<BF16>();
            if (item < n) raw[i] = piece_load<BF16>(H, item * ldh + (p % PPR) * 8);
        }
    };
    auto stash = [&](int64_t stage, int in_unit, unsigned parity) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int p = i * 256 + tid, row = p / PPR;
            *(bf16x8 *)(lds[stage & 1] + row * PITCH + (p % PPR) * 16) = piece_bf16<BF16>(raw[i]);
            if (with_norms) {
                float x[8], ss = 0.f, am = 0.f;
                piece_floats<BF16>(raw[i], x);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    ss = fmaf(x[e], x[e], ss);
                    am = fmaxf(am, fabsf(x[e]));
                }
                ss = group_reduce<PPR>(ss, [](float u, float v) { return u + v; });
                am = group_reduce<PPR>(am, [](float u, float v) { return fmaxf(u, v); });
                if (p % PPR == 0) atomicMax(&nmax[parity][((in_unit * S + row) / TOPK_SEG) & 3], __float_as_uint(norm_bound(ss, am, D)));
            }
        }
    };

    float best[NM][QT];
    auto reset = [&] {
#pragma unroll
        for (int c = 0; c < NM; ++c)
#pragma unroll
            for (int t = 0; t < QT; ++t) best[c][t] = -INFINITY;
    };
    reset();
    if (tid < 8) nmax[tid >> 2][tid & 3] = 0u;
    fetch(0);
    __syncthreads();
    stash(0, 0, 0);
    __syncthreads();
    int64_t unit = u0;
    for (int64_t st = 0, in_unit = 0; st < stages; ++st) {
        if (st + 1 < stages) fetch(st + 1);
        const char *rows = lds[st & 1];
#pragma unroll
        for (int i = 0; i < SUB; ++i) {
            const char *mine = rows + ((WI == 1 ? i : wave) * TOPK_SEG + a) * PITCH + h * 16;
            floatx16 acc[QT];
#pragma unroll
            for (int t = 0; t < QT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 ah = *(const bf16x8 *)(mine + s * 32);
#pragma unroll
                for (int t = 0; t < QT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bq[t][s], acc[t], 0, 0, 0);
            }
            // acc[t][v] = <query 32 t + a, item 8 (v / 4) + 4 h + v % 4 of the segment>
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                float m = best[i % NM][t];
#pragma unroll
                for (int v = 0; v < 16; v += 2) m = fmaxf(fmaxf(m, acc[t][v]), acc[t][v + 1]);
                best[i % NM][t] = m;
            }
        }
        if constexpr (WI == 1 && SUB == 2) {  // the next stage holds segments of the unit's other two chunks
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                const float x = best[0][t], y = best[1][t];
                best[0][t] = best[2][t]; best[1][t] = best[3][t];
                best[2][t] = x; best[3][t] = y;
            }
        }
        const bool unit_done = ++in_unit == spu;
        if (unit_done) {
            in_unit = 0;
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                float m[NM];
#pragma unroll
                for (int c = 0; c < NM; ++c) m[c] = fmaxf(best[c][t], __shfl_xor(best[c][t], 32));
                if (h == 0 && query[t] < nq) {
                    if constexpr (WI == 1) *(float4 *)(maxima + maxima_at((int)(4 * unit), query[t], nq)) = make_float4(m[0], m[1], m[2], m[3]);
                    else maxima[maxima_at((int)(4 * unit) + wave, query[t], nq)] = m[0];
                }
            }
            reset();
            if (with_norms && tid < 4) {
                // every row of this unit was entered before the last barrier; the slot is used again two units on
                const unsigned par = (unsigned)(unit - u0) & 1;
                norms[4 * unit + tid] = __uint_as_float(nmax[par][tid]);
                nmax[par][tid] = 0u;
            }
            ++unit;
        }
        if (st + 1 < stages) stash(st + 1, (int)in_unit, (unsigned)(unit - u0) & 1);
        __syncthreads();
    }
}

__device__ __forceinline__ bool ranks_before(float sa, int32_t ia, float sb, int32_t ib) {
    return sa > sb || (sa == sb && ia < ib);
}

// Bitonic sort of N (a power of two) candidates in LDS by the whole workgroup, best first.
__device__ __forceinline__ void block_sort(float *sc, int32_t *id, int N, int tid) {
    for (int k2 = 2; k2 <= N; k2 <<= 1) {
        for (int j = k2 >> 1; j > 0; j >>= 1) {
            for (int t = tid; t < N / 2; t += 256) {
                const int i = (t & ~(j - 1)) * 2 + (t & (j - 1)), l = i + j;
                const float sa = sc[i], sb = sc[l];
                const int32_t ia = id[i], ib = id[l];
                const bool first_i = (i & k2) == 0;  // this block is sorted best-first / best-last
                if (ranks_before(sb, ib, sa, ia) == first_i) {
                    sc[i] = sb; sc[l] = sa;
                    id[i] = ib; id[l] = ia;
                }
            }
            __syncthreads();
        }
    }
}

// Full-accuracy scores of 16 queries and 16 items: bf16 rows of 32 elements and more as they are stored on the bf16 matrix
// cores (exact products, fp32 sums), everything else as fp32 on v_mfma_f32_16x16x4f32, which rounds every product's sum to
// nearest.  The order of the sums is fixed, 16 or 32 elements per round of matrix instructions: it decides which of two items
// whose scores differ by less than their rounding comes first, so a score has the same bits wherever it is computed.  Lane
// (a, q) = (lane % 16, lane / 16) holds, of query a and of item a, the 16-byte pieces j of the row: elements (4 j + q) EPP ..
template <int D, bool BF16> constexpr bool score_native() { return BF16 && D >= 32; }
template <int D, bool BF16> constexpr int score_pieces() { return D / (score_native<D, BF16>() ? 32 : 16); }
template <int D, bool BF16>
__device__ __forceinline__ void score_load(const void *T, int64_t elem0, bool ok, int q, float4 (&z)[score_pieces<D, BF16>()]) {
    constexpr int NP = score_pieces<D, BF16>();
#pragma unroll
    for (int j = 0; j < NP; ++j) z[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ok) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            if constexpr (score_native<D, BF16>()) {
                z[j] = *(const float4 *)((const uint16_t *)T + elem0 + (4 * j + q) * 8);
            } else {
                float x[4];
                load_vec<4, BF16>(T, elem0 + (4 * j + q) * 4, x);
                z[j] = make_float4(x[0], x[1], x[2], x[3]);
            }
        }
    }
}
// element v of lane (a, q): <query 4 q + v, item a>
template <int D, bool BF16>
__device__ __forceinline__ floatx4 score_tile(const float4 (&zq)[score_pieces<D, BF16>()], const float4 (&zh)[score_pieces<D, BF16>()]) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < score_pieces<D, BF16>(); ++j) {
        if constexpr (score_native<D, BF16>()) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, zq[j]), __builtin_bit_cast(bf16x8, zh[j]), acc, 0, 0, 0);
        } else {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(zq[j].x, zh[j].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(zq[j].y, zh[j].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(zq[j].z, zh[j].z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(zq[j].w, zh[j].w, acc, 0, 0, 0);
        }
    }
    return acc;
}

// What bounds it: the latency of its few dependent phases (maxima, rescoring, sort) when there are few queries, the read
// of the maxima and of the rescored chunks when there are many.
// Rescoring takes two forms.  bf16 rows of 32 elements and more go through score_tile at once.  The fp32 matrix instruction,
// of which fifteen sixteenths are idle here, would bound the kernel: such rows are first scored by eight products per lane and
// a sum over lanes, and only the items that this does not rule out (its rounding allowed for) go through score_tile, 16 at a
// time (every item through it / as it is: 4096 x 10M fp32, d = 128, k = 20: 29.6 / 20.4 ms, 64 x 30k, d = 64: 38 / 36 us).
// Both kernels together against a scan that scored everything in full and kept candidate buffers: 64 queries x 30k items
// (d = 64, fp32, k = 20) 2.36 -> 0.036 ms, 4096 x 1M (the same) 7.9 -> 0.82 ms, 4096 x 10M (d = 128, bf16, k = 50,
// exclusions) 131 -> 10.4 ms.
template <int D, bool BF16>
__global__ __launch_bounds__(TOPK_SELECT_THREADS) void topk_select_kernel(const void *__restrict__ Q, int64_t ldq, int64_t nq,
                                                          const void *__restrict__ H, int64_t ldh, int64_t n,
                                                          const int64_t *__restrict__ ex_indptr,
                                                          const int32_t *__restrict__ ex_indices, int k, ChunkMap map,
                                                          const float *__restrict__ maxima, const float *__restrict__ norms,
                                                          int32_t *__restrict__ deferred, int defer_chunks,
                                                          int32_t *__restrict__ ids, float *__restrict__ scores) {
    constexpr int LPI = D / 8, IPS = 64 / LPI, STEPS = TOPK_SEG / IPS;  // lanes per item, items per step and wavefront
    constexpr int NP = score_pieces<D, BF16>();
    constexpr bool NATIVE = score_native<D, BF16>();
    constexpr int32_t NO_ID = 0x7fffffff;
    extern __shared__ uint32_t touched[];  // one bit per chunk: it holds an excluded item
    __shared__ float tmax[256], sc[TOPK_CAND], list_u[TOPK_LIST];
    __shared__ int32_t id[TOPK_CAND], list_c[TOPK_LIST];
    __shared__ int count, nlist, bar_id;
    __shared__ float bar;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t q = blockIdx.x;
    const int64_t eb = ex_indptr ? ex_indptr[q] : 0, ee = ex_indptr ? ex_indptr[q + 1] : 0;

    float4 zq[NATIVE ? NP : 1];
    if constexpr (NATIVE) score_load<D, BF16>(Q, q * ldq, true, lane >> 4, zq);
    float qx[8];  // this lane's eight elements of the query
    piece_floats<BF16>(piece_load<BF16>(Q, q * ldq + (lane % LPI) * 8), qx);
    float ss = 0.f, am = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ss = fmaf(qx[e], qx[e], ss);
        am = fmaxf(am, fabsf(qx[e]));
    }
    ss = group_reduce<LPI>(ss, [](float u, float v) { return u + v; });
    am = group_reduce<LPI>(am, [](float u, float v) { return fmaxf(u, v); });
    const float qn = norm_bound(ss, am, D);

    if (ee > eb) {
        for (int w = tid; w < (map.nchunks + 31) / 32; w += 256) touched[w] = 0u;
        __syncthreads();
        for (int64_t p = eb + tid; p < ee; p += 256) {
            const int64_t e = ex_indices[p];
            if (e >= 0 && e < n) {
                const int c = map.of_item(e);
                atomicOr(&touched[c >> 5], 1u << (c & 31));
            }
        }
    }
    if (tid == 0) {
        count = nlist = 0;
        bar = -INFINITY;
        bar_id = NO_ID;
    }
    __syncthreads();

    // the bar: k-th largest of the threads' best lower bounds (different chunks, so different items)
    float low = -INFINITY, high = -INFINITY;
    bool unbounded = false;
    for (int c0 = 4 * tid; c0 < map.nchunks; c0 += 1024) {
        const float4 m4 = *(const float4 *)(maxima + maxima_at(c0, q, nq)), n4 = *(const float4 *)(norms + c0);
        const float m[4] = {m4.x, m4.y, m4.z, m4.w}, nn[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float g = margin<D, BF16>(qn, nn[j]);
            const bool dirty = ee > eb && ((touched[(c0 + j) >> 5] >> ((c0 + j) & 31)) & 1u);
            if (g < INFINITY) {
                high = fmaxf(high, m[j] + g);
                if (!dirty && map.complete(c0 + j, n)) low = fmaxf(low, m[j] - g);
            } else {
                unbounded = true;
            }
        }
    }
    tmax[tid] = low;
    __syncthreads();
    int rank = 0;
    for (int t = 0; t < 256; t += 4) {
        const float4 o4 = *(const float4 *)(tmax + t);
        const float o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) rank += o[j] > low || (o[j] == low && t + j < tid);
    }
    if (rank == k - 1) bar = low;
    __syncthreads();

    // chunk c may hold one of the best k: its upper bound reaches the bar (equal scores rank by id)
    auto scan4 = [&](int c0) {
        const float4 m4 = *(const float4 *)(maxima + maxima_at(c0, q, nq)), n4 = *(const float4 *)(norms + c0);
        const float m[4] = {m4.x, m4.y, m4.z, m4.w}, nn[4] = {n4.x, n4.y, n4.z, n4.w};
        const float b = bar;
        const int32_t bi = bar_id;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float g = margin<D, BF16>(qn, nn[j]);
            const float u = g < INFINITY ? m[j] + g : INFINITY;
            const int64_t first = map.first(c0 + j);
            if (first < n && !(u < b) && !(u == b && first > bi)) {
                const int pos = atomicAdd(&nlist, 1);
                if (pos < TOPK_LIST) {
                    list_c[pos] = c0 + j;
                    list_u[pos] = u;
                }
            }
        }
    };
    // sort the candidates, keep the best k, raise the bar
    auto cut = [&] {
        const int c = count;
        int N = 2;
        while (N < c) N <<= 1;
        for (int t = c + tid; t < N; t += 256) {
            sc[t] = -INFINITY;
            id[t] = NO_ID;
        }
        __syncthreads();
        block_sort(sc, id, N, tid);
        if (tid == 0 && c > k) count = k;
        if (tid == 0 && c >= k && id[k - 1] != NO_ID) {
            bar = sc[k - 1];
            bar_id = id[k - 1];
        }
        __syncthreads();
    };
    // full-accuracy scores of the listed chunks, one segment per wavefront and step
    auto rescore = [&](int listed) {
        const int lr = map.lc - 5, total = listed << lr;
        for (int base = 0; base < total; base += 4 * TOPK_ROUND) {
            if (count + 4 * TOPK_ROUND * TOPK_SEG > TOPK_CAND) cut();
            const int before = count;
            const float b = bar;
            const int32_t bi = bar_id;
            __syncthreads();
            for (int r = 0; r < TOPK_ROUND; ++r) {
                const int g = base + 4 * r + wave;
                if (g >= total) break;
                const int64_t i0 = map.segment(list_c[g >> lr], g & ((1 << lr) - 1));
                const float u = list_u[g >> lr];
                if (u < b || (u == b && i0 > bi)) continue;
                if constexpr (NATIVE) {
                    float4 z[2][NP];
                    floatx4 acc[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) score_load<D, BF16>(H, (i0 + 16 * t + (lane & 15)) * ldh, i0 + 16 * t + (lane & 15) < n, lane >> 4, z[t]);
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[t] = score_tile<D, BF16>(zq, z[t]);
                    const float v = lane < 16 ? acc[0][0] : acc[1][0];  // every row of a tile is this query
                    const int64_t item = i0 + lane;
                    if (lane < TOPK_SEG && item < n && (v > b || (v == b && (int32_t)item < bi))) {
                        const int pos = atomicAdd(&count, 1);  // a round adds at most 4 * TOPK_ROUND * TOPK_SEG
                        sc[pos] = v;
                        id[pos] = (int32_t)item;
                    }
                } else {
                    // the order of a score's sums does not matter yet: both are within `slack` of each other
                    const float slack = margin<D, true>(qn, norms[list_c[g >> lr]]);
                    Piece<BF16> p[STEPS];
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) {
                        const int64_t item = i0 + s * IPS + lane / LPI;
                        p[s] = piece_zero<BF16>();
                        if (item < n) p[s] = piece_load<BF16>(H, item * ldh + (lane % LPI) * 8);
                    }
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) {
                        const int64_t item = i0 + s * IPS + lane / LPI;
                        float x[8], v = 0.f;
                        piece_floats<BF16>(p[s], x);
#pragma unroll
                        for (int e = 0; e < 8; ++e) v = fmaf(qx[e], x[e], v);
                        v = group_reduce<LPI>(v, [](float u, float w) { return u + w; });
                        if (lane % LPI == 0 && item < n && !(v + slack < b)) id[atomicAdd(&count, 1)] = (int32_t)item;
                    }
                }
            }
            __syncthreads();
            const int after = count;
            if constexpr (!NATIVE) {
                for (int t0 = before + 16 * wave; t0 < after; t0 += 64) {
                    const int t = t0 + (lane & 15);
                    const int32_t item = t < after ? id[t] : 0;
                    float4 zq[NP], z[NP];
                    score_load<D, BF16>(Q, q * ldq, true, lane >> 4, zq);
                    score_load<D, BF16>(H, item * ldh, t < after, lane >> 4, z);
                    const float v = score_tile<D, BF16>(zq, z)[0];  // every row of the tile is this query
                    if (lane < 16 && t < after) {
                        const bool keep = v > b || (v == b && item < bi);
                        sc[t] = keep ? v : -INFINITY;
                        if (!keep) id[t] = NO_ID;
                    }
                }
                if (after > before) __syncthreads();
            }
            if (after > before && ee > eb) {
                for (int64_t p = eb + tid; p < ee; p += 256) {
                    const int32_t e = ex_indices[p];
                    for (int t = before; t < after; ++t) {
                        if (id[t] == e) {
                            sc[t] = -INFINITY;
                            id[t] = NO_ID;
                        }
                    }
                }
                __syncthreads();
            }
        }
    };

    // Usually the list holds everything that is left: only threads whose best upper bound reaches the bar look again.
    if (unbounded || !(high < bar))
        for (int c0 = 4 * tid; c0 < map.nchunks; c0 += 1024) scan4(c0);
    __syncthreads();
    const int found = nlist;
    if (found > defer_chunks) {  // the scan takes this query
        if (tid == 0) deferred[1 + atomicAdd(&deferred[0], 1)] = (int32_t)q;
        return;
    }
    if (found <= TOPK_LIST) {
        rescore(found);
    } else {  // ties or values without a bound: 1024 chunks at a time, the bar rising between
        for (int base = 0; base < map.nchunks; base += 1024) {
            __syncthreads();
            if (tid == 0) nlist = 0;
            __syncthreads();
            if (base + 4 * tid < map.nchunks) scan4(base + 4 * tid);
            __syncthreads();
            rescore(nlist);
        }
    }
    cut();
    if (tid < k) {
        const bool have = tid < count && id[tid] != NO_ID;
        ids[q * k + tid] = have ? id[tid] : -1;
        scores[q * k + tid] = have ? sc[tid] : -INFINITY;
    }
}

// Bitonic sort of N (a power of two) candidates in LDS by one wavefront, best first.
template <int N> __device__ __forceinline__ void wave_sort(float *sc, int32_t *id, int lane) {
    for (int k2 = 2; k2 <= N; k2 <<= 1) {
        for (int j = k2 >> 1; j > 0; j >>= 1) {
            for (int t = lane; t < N / 2; t += 64) {
                const int i = (t / j) * 2 * j + (t % j), l = i + j;
                const float sa = sc[i], sb = sc[l];
                const int32_t ia = id[i], ib = id[l];
                const bool first_i = (i & k2) == 0;  // this block is sorted best-first / best-last
                if (ranks_before(sb, ib, sa, ia) == first_i) {
                    sc[i] = sb; sc[l] = sa;
                    id[i] = ib; id[l] = ia;
                }
            }
            wave_sync();
        }
    }
}

// What bounds it: the latency of one round after the other for few queries, the fp32 matrix instruction for many.
// deferred[0] queries are left to it (none, usually: the workgroups return at once), deferred[1 + x] is the x-th; its
// slice y leaves its candidates at [y * nq + x].
template <int D, bool BF16>
__global__ __launch_bounds__(64 * SCAN_WAVES) void topk_scan_kernel(
    const void *__restrict__ Q, int64_t ldq, int64_t nq, const void *__restrict__ H, int64_t ldh, int64_t n,
    const int64_t *__restrict__ ex_indptr, const int32_t *__restrict__ ex_indices, int k, int kpad,
    int64_t slice_items, const int32_t *__restrict__ deferred, float *__restrict__ part_sc, int32_t *__restrict__ part_id) {
    extern __shared__ float lds[];
    constexpr int NP = score_pieces<D, BF16>();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, a = lane & 15, q = lane >> 4;
    // per wavefront: scores [16][CAP], ids [16][CAP], count [16], bar [16]
    float *sc = lds + wave * (2 * SCAN_QPW * SCAN_CAP + 2 * SCAN_QPW);
    int32_t *id = (int32_t *)(sc + SCAN_QPW * SCAN_CAP);
    int32_t *cnt = id + SCAN_QPW * SCAN_CAP;
    float *bar = (float *)(cnt + SCAN_QPW);
    const int64_t todo = deferred[0];
    const int64_t q0 = ((int64_t)blockIdx.x * SCAN_WAVES + wave) * SCAN_QPW;
    if (q0 >= todo) return;  // wavefronts are independent of each other: no workgroup barrier below
    if (lane < SCAN_QPW) {
        cnt[lane] = 0;
        bar[lane] = -INFINITY;
    }
    float4 zq[NP];
    score_load<D, BF16>(Q, q0 + a < todo ? deferred[1 + q0 + a] * ldq : 0, q0 + a < todo, q, zq);
    wave_sync();
    const int64_t i0 = (int64_t)blockIdx.y * slice_items, i1 = i0 + slice_items < n ? i0 + slice_items : n;

    auto compact = [&](int qy) {  // sort query qy's buffer, keep its best k, raise its bar
        float *s = sc + qy * SCAN_CAP;
        int32_t *d = id + qy * SCAN_CAP;
        const int c = cnt[qy];
        for (int t = c + lane; t < SCAN_CAP; t += 64) {
            s[t] = -INFINITY;
            d[t] = 0x7fffffff;
        }
        wave_sync();
        wave_sort<SCAN_CAP>(s, d, lane);
        if (lane == 0) {
            const int keep = c < k ? c : k;
            cnt[qy] = keep;
            bar[qy] = keep == k ? s[k - 1] : -INFINITY;
        }
        wave_sync();
    };

    // SCAN_TILES tiles of 16 items per round; the next round's rows are requested before this round's products
    float4 zh[SCAN_TILES][NP], zn[SCAN_TILES][NP];
#pragma unroll
    for (int u = 0; u < SCAN_TILES; ++u) score_load<D, BF16>(H, (i0 + 16 * u + a) * ldh, i0 + 16 * u + a < i1, q, zh[u]);
    for (int64_t t0 = i0; t0 < i1; t0 += 16 * SCAN_TILES) {
#pragma unroll
        for (int u = 0; u < SCAN_TILES; ++u) {
            const int64_t nxt = t0 + 16 * (SCAN_TILES + u) + a;
            score_load<D, BF16>(H, nxt * ldh, nxt < i1, q, zn[u]);
        }
        floatx4 acc[SCAN_TILES];
#pragma unroll
        for (int u = 0; u < SCAN_TILES; ++u) acc[u] = score_tile<D, BF16>(zq, zh[u]);
        // acc[u][v] = <query q0 + 4q + v, item t0 + 16 u + a>
        const float4 b4 = *(const float4 *)(bar + 4 * q);
        const float bq[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int u = 0; u < SCAN_TILES; ++u) {
            const int64_t item = t0 + 16 * u + a;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int qy = 4 * q + v;
                if (item < i1 && q0 + qy < todo && acc[u][v] >= bq[v]) {
                    bool skip = false;
                    if (ex_indptr) {
                        const int64_t row = deferred[1 + q0 + qy], eb = ex_indptr[row], ee = ex_indptr[row + 1];
                        for (int64_t p = eb; p < ee; ++p) skip |= ex_indices[p] == (int32_t)item;
                    }
                    if (!skip) {
                        const int pos = atomicAdd(&cnt[qy], 1);  // at most 16 per tile and query: never beyond CAP
                        sc[qy * SCAN_CAP + pos] = acc[u][v];
                        id[qy * SCAN_CAP + pos] = (int32_t)item;
                    }
                }
            }
        }
        wave_sync();
        const int mine = lane < SCAN_QPW ? cnt[lane] : 0;
        unsigned long long full = __ballot(mine > SCAN_CAP - 16 * SCAN_TILES);
        while (full) {
            const int qy = __ffsll((long long)full) - 1;
            full &= full - 1;
            compact(qy);
        }
#pragma unroll
        for (int u = 0; u < SCAN_TILES; ++u)
#pragma unroll
            for (int j = 0; j < NP; ++j) zh[u][j] = zn[u][j];
    }
    for (int qy = 0; qy < SCAN_QPW; ++qy) {
        compact(qy);
        if (q0 + qy < todo && lane < kpad) {
            const int64_t o = ((int64_t)blockIdx.y * nq + q0 + qy) * kpad + lane;
            const bool have = lane < cnt[qy];
            part_sc[o] = have ? sc[qy * SCAN_CAP + lane] : -INFINITY;
            part_id[o] = have ? id[qy * SCAN_CAP + lane] : 0x7fffffff;
        }
    }
}

// One wavefront per deferred query: the slices' candidates, sorted, best k written (ids -1 and scores -inf where the
// table has fewer than k admissible rows).
__global__ __launch_bounds__(64) void topk_merge_kernel(const float *__restrict__ part_sc,
                                                        const int32_t *__restrict__ part_id, int64_t nq, int slices,
                                                        int kpad, int k, const int32_t *__restrict__ deferred,
                                                        int32_t *__restrict__ ids, float *__restrict__ scores) {
    __shared__ float sc[SCAN_MERGE];
    __shared__ int32_t id[SCAN_MERGE];
    const int lane = threadIdx.x;
    if ((int64_t)blockIdx.x >= deferred[0]) return;
    const int64_t row = deferred[1 + blockIdx.x];
    const int total = slices * kpad;
    for (int t = lane; t < SCAN_MERGE; t += 64) {
        float s = -INFINITY;
        int32_t d = 0x7fffffff;
        if (t < total) {
            const int64_t o = ((int64_t)(t / kpad) * nq + blockIdx.x) * kpad + t % kpad;
            s = part_sc[o];
            d = part_id[o];
        }
        sc[t] = s;
        id[t] = d;
    }
    wave_sync();
    wave_sort<SCAN_MERGE>(sc, id, lane);
    if (lane < k) {
        const bool have = id[lane] != 0x7fffffff;
        ids[row * k + lane] = have ? id[lane] : -1;
        scores[row * k + lane] = have ? sc[lane] : -INFINITY;
    }
}

template <int D, bool BF16, int QT, int WI>
static void bound_launch(const als_ctx *ctx, const void *Q, int64_t ldq, int64_t nq, const als_table *H, ChunkMap map,
                         float *maxima, float *norms, int32_t *deferred, hipStream_t s) {
    const int64_t gq = topk_group_queries<QT, WI>(), qgroups = (nq + gq - 1) / gq, units = map.nchunks / 4;
    // 32 workgroups per compute unit where the table has them: the workgroups of one item stretch stay close in time, so
    // their reads meet in L2 (4096 queries x 10M items, d = 128, bf16: 10.9 ms with 8 per unit, 10.45 with 32, 10.5 with 64)
    const int64_t want = std::max<int64_t>(1, (int64_t)ctx->num_cu * 32 / qgroups);
    const int64_t per = std::max<int64_t>(1, (units + want - 1) / want), splits = (units + per - 1) / per;
    const unsigned blocks = (unsigned)((splits + 7) / 8 * 8 * qgroups);
    hipLaunchKernelGGL((topk_bound_kernel<D, BF16, QT, WI>), dim3(blocks), dim3(256), 0, s, Q, ldq, nq, H->data, H->ld, H->rows,
                       map, (unsigned)qgroups, per, maxima, norms, deferred);
}

template <int D, bool BF16>
static als_status topk_typed(als_ctx *ctx, const als_table *Q, const als_table *H, const als_csr *ex, int k,
                             int32_t *ids, float *scores, hipStream_t s) {
    constexpr int64_t ES = BF16 ? 2 : 4;
    // Chunk size: a chunk costs 12 bytes of maxima per query (written once, read twice) and the matrix cores' pause at its
    // end, rescoring about 1.3 k chunks of C rows each; C^2 = 48 n / (1.3 k row bytes) balances them.  Measured at the size
    // this gives, half and twice of it: 0.79, 0.95, 0.85 ms (4096 x 1M, d = 64, fp32, k = 20), 10.45, 12.1, 10.7 ms
    // (4096 x 10M, d = 128, bf16, k = 50).
    ChunkMap map{5, 0};
    const double best2 = 48.0 * (double)H->rows / (1.3 * k * D * ES);
    while (map.lc < 24 && (std::exp2(2 * map.lc + 1) < best2 || (H->rows >> map.lc) >= TOPK_MAX_CHUNKS)) ++map.lc;
    map.nchunks = (int)(4 * ((H->rows + map.unit_items() - 1) / map.unit_items()));
    // A query is left to the scan when more than 1/16 of the chunks reach its bar (and more than eight times what k items in
    // different chunks need, on small tables).  Alone, one workgroup walks a table at about 30 GB/s and a chip full of them at
    // 8 TB/s, while the scan takes as long for one query as for some hundred.  Nearly parallel rows, every query by itself
    // to the end / left to the scan / a scan from the start (d = 64, fp32, k = 20): 4096 x 1M 133 / 9.0 / 8.0 ms,
    // 1024 x 1M 29 / 2.5 / 2.1 ms, 1 x 1M 8.8 / 1.4 / 1.3 ms, 8192 x 30k 3.4 / 1.08 / 0.91 ms, 64 x 30k 0.36 / - / 0.52 ms.
    // Small calls and tables, where walking alone is the shorter, are spared the scan's two launches (about 5 us when no
    // query needs them).
    const double table_bytes = (double)H->rows * D * ES;
    const int many_chunks = std::max(map.nchunks / 16, 8 * k);
    const bool may_scan = many_chunks < map.nchunks &&
                          (table_bytes >= (double)(1 << 24) || table_bytes * (double)Q->rows >= 4294967296.0);
    const int defer_chunks = may_scan ? many_chunks : INT32_MAX;
    int kpad = 1;
    while (kpad < k) kpad <<= 1;
    int slices = (int)std::min<int64_t>(SCAN_MERGE / kpad, std::max<int64_t>(1, (H->rows + 8191) / 8192));
    const int64_t slice_items = ((H->rows + slices - 1) / slices + 15) / 16 * 16;
    if (may_scan) slices = (int)((H->rows + slice_items - 1) / slice_items);
    // Queries go in batches whose maxima and partial lists fit TOPK_BATCH_BYTES; each batch reads the item table once more.
    constexpr int64_t TOPK_BATCH_BYTES = (int64_t)3 << 29;
    const int64_t maxima_bytes = (map.nchunks + 15) / 16 * 16 * (int64_t)sizeof(float);
    const int64_t scan_bytes = may_scan ? (int64_t)slices * kpad * (int64_t)(sizeof(float) + sizeof(int32_t)) : 0;
    const int64_t per_query = std::max(maxima_bytes, scan_bytes);  // the scan's partial lists lie where the maxima were
    constexpr int QT = D == 128 ? 3 : 4;
    const size_t norm_bytes = ((size_t)map.nchunks * sizeof(float) + 255) / 256 * 256;
    size_t defer_bytes = 0;
    int64_t batch = topk_batch(Q->rows, per_query, topk_group_queries<QT, 1>(), TOPK_BATCH_BYTES);
    for (const std::string last = ctx->last_error;;) {
        defer_bytes = ((size_t)(batch + 1) * sizeof(int32_t) + 255) / 256 * 256;
        const als_status st = ensure(ctx, ctx->topk_partials, norm_bytes + defer_bytes + (size_t)(batch * per_query));
        if (st == ALS_OK) {
            ctx->last_error = last;
            break;
        }
        const int64_t less = topk_smaller_batch(batch);  // a nearly full card: the table is read more often
        if (st != ALS_ENOMEM || less == batch) return st;
        batch = less;
    }
    float *norms = (float *)ctx->topk_partials.p, *maxima = (float *)((char *)ctx->topk_partials.p + norm_bytes + defer_bytes);
    int32_t *deferred = (int32_t *)((char *)ctx->topk_partials.p + norm_bytes);
    float *part_sc = maxima;
    int32_t *part_id = (int32_t *)(part_sc + (size_t)slices * batch * kpad);
    const size_t bitmap = ex ? ((size_t)map.nchunks + 31) / 32 * 4 : 0;
    constexpr int scan_lds = SCAN_WAVES * (2 * SCAN_QPW * SCAN_CAP + 2 * SCAN_QPW) * 4;
    static const hipError_t attr = hipFuncSetAttribute((const void *)topk_scan_kernel<D, BF16>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, scan_lds);  // once per process
    ALS_HIP(ctx, attr);
    for (int64_t q0 = 0; q0 < Q->rows; q0 += batch) {
        const int64_t nq = std::min(batch, Q->rows - q0);
        const void *Qb = (const char *)Q->data + q0 * Q->ld * ES;
        const int64_t *ex_ptr = ex ? ex->indptr + q0 : nullptr;
        const int32_t *ex_idx = ex ? ex->indices : nullptr;
        if (map.nchunks > 0) {
            if (nq <= 256) bound_launch<D, BF16, 2, 4>(ctx, Qb, Q->ld, nq, H, map, maxima, norms, deferred, s);
            else bound_launch<D, BF16, QT, 1>(ctx, Qb, Q->ld, nq, H, map, maxima, norms, deferred, s);
        }
        hipLaunchKernelGGL((topk_select_kernel<D, BF16>), dim3((unsigned)nq), dim3(TOPK_SELECT_THREADS), bitmap, s, Qb, Q->ld, nq, H->data,
                           H->ld, H->rows, ex_ptr, ex_idx, k, map, (const float *)maxima, (const float *)norms, deferred,
                           defer_chunks, ids + q0 * k, scores + q0 * k);
        if (may_scan) {
            const unsigned groups = (unsigned)((nq + SCAN_QPW * SCAN_WAVES - 1) / (SCAN_QPW * SCAN_WAVES));
            hipLaunchKernelGGL((topk_scan_kernel<D, BF16>), dim3(groups, slices), dim3(64 * SCAN_WAVES), scan_lds, s, Qb, Q->ld,
                               nq, H->data, H->ld, H->rows, ex_ptr, ex_idx, k, kpad, slice_items, (const int32_t *)deferred,
                               part_sc, part_id);
            hipLaunchKernelGGL(topk_merge_kernel, dim3((unsigned)nq), dim3(64), 0, s, (const float *)part_sc,
                               (const int32_t *)part_id, nq, slices, kpad, k, (const int32_t *)deferred, ids + q0 * k,
                               scores + q0 * k);
        }
    }
    ALS_HIP(ctx, hipGetLastError());
    return ALS_OK;
}

als_status launch_topk(als_ctx *ctx, const als_table *Q, const als_table *H, const als_csr *ex, int k, int32_t *ids,
                       float *scores, hipStream_t s) {
    const bool bf = H->dtype == ALS_BF16;
    switch (H->d) {
        case 16: return bf ? topk_typed<16, true>(ctx, Q, H, ex, k, ids, scores, s) : topk_typed<16, false>(ctx, Q, H, ex, k, ids, scores, s);
        case 32: return bf ? topk_typed<32, true>(ctx, Q, H, ex, k, ids, scores, s) : topk_typed<32, false>(ctx, Q, H, ex, k, ids, scores, s);
        case 64: return bf ? topk_typed<64, true>(ctx, Q, H, ex, k, ids, scores, s) : topk_typed<64, false>(ctx, Q, H, ex, k, ids, scores, s);
        case 128: return bf ? topk_typed<128, true>(ctx, Q, H, ex, k, ids, scores, s) : topk_typed<128, false>(ctx, Q, H, ex, k, ids, scores, s);
    }
    return fail(ctx, ALS_EDTYPE, "unsupported d");
}

}  // namespace als
