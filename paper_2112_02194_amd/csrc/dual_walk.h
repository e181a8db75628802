// Walking the list of a row class that is worked four rows per step and wavefront.
#pragma once

#include "dual_common.h"
#include "x_rows.h"

namespace als {

// The four rows of step `blk` (4 blk < count), wavefront-uniform: row relative to r0 (-1 past the end of the list, with k = 0
// and the step's first row's b), first entry, entries.
struct RowsRel { int32_t rel[4]; };
struct RowsDesc {
    RowsRel row;
    int64_t b[4];
    int k[4];
};
__device__ __forceinline__ RowsRel rows_rel(const int32_t *__restrict__ list, int count, int blk) {
    // one 16-byte read of the four list entries (the list's workspace is padded for it)
    const ListQuad r4 = *(const ListQuad *)(list + (int64_t)blk * 4);
    const int first = blk * 4;
    return {{r4.x, first + 1 < count ? r4.y : r4.x, first + 2 < count ? r4.z : r4.x, first + 3 < count ? r4.w : r4.x}};
}
struct RowsBounds { int64_t b[4], e[4]; };
__device__ __forceinline__ RowsBounds rows_bounds(const int64_t *__restrict__ indptr, int64_t r0, const RowsRel &rel) {
    RowsBounds w;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        w.b[p] = indptr[r0 + rel.rel[p]];
        w.e[p] = indptr[r0 + rel.rel[p] + 1];
    }
    return w;
}
__device__ __forceinline__ RowsDesc rows_desc(const RowsRel &rel, RowsBounds w, int count, int blk) {
    RowsDesc d;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        asm volatile("" : "+s"(w.b[p]), "+s"(w.e[p]));  // loaded whether the row exists or not: no branch around the loads
        const bool have = blk * 4 + p < count;
        d.row.rel[p] = have ? rel.rel[p] : -1;
        d.b[p] = w.b[p];
        d.k[p] = have ? (int)(w.e[p] - w.b[p]) : 0;
    }
    return d;
}

// Ids are waited for here: left to their first use, the wait comes behind loads and stores issued in between and takes them in.
template <int N> __device__ __forceinline__ void wait_ids(int32_t (&idv)[N]) {
#pragma unroll
    for (int n = 0; n < N; ++n) asm volatile("" : "+v"(idv[n]));
}

// A step type S provides
//   NIDS, ids(indices, desc, lane, idv)   the column ids that a lane holds
//   init(lds, lane)                       once per wavefront
//   solve(values, Z, err_flag, lds, desc, idv, loaded, between, last, out)
//         one step; calls `loaded` when the loads of the entries are under way, `between` once the entries have been used for S,
//         before the elimination, `last` before it gives away its rows: out.store<lanes of a row>(rv, lane), see store_rows
//   FREE  offset in LDS of a place for four rows of R that is free when the rows are given away (steps that Parked is used with)

// rows of a step to R
struct RowsOut {
    float *R;
    int64_t ldr;
    const RowsRel &row;
    template <int LPR, int NV> __device__ __forceinline__ void store(const floatx4 (&rv)[4][NV], int lane) const {
        const int64_t u[4] = {row.rel[0], row.rel[1], row.rel[2], row.rel[3]};
        store_rows<LPR>(rv, R, ldr, u, lane);
    }
    template <int LPR, int NV> __device__ __forceinline__ void store_one(const floatx4 (&rv)[NV], int lane) const {
        store_row<LPR>(rv, R + row.rel[0] * ldr, lane);
    }
};

// Rows of up to four steps kept in LDS until x_rows_from_memory takes sixteen of them at a time: X = R L^-1 for bf16 tables.  Three
// steps have places behind the step's own LDS, the fourth takes the place that the step names as free.  (A wavefront has about four steps.)
// The matrix, 40 KB at d = 128, comes from the L2: there is no room in LDS beside eight wavefronts of 16 < k <= 32.
// Epoch of 50M x 50M power-law rows (d = 128): 211.4 -> 201.3 ms (16 < k <= 32 72.3 -> 74.6 ms, 8 < k <= 16 23.9 -> 23.8, the pass over the rows
// left 16.8 -> 1.6; 76.2, 25.0 with the matrix loads left to the compiler).
struct XTable {
    uint16_t *X;      // row r0
    int64_t ldx;
    const char *mat;  // XMatrix<D, true>, in device memory
};
template <class S, int D> struct Parked {
    static constexpr int RLD = D + 4, OFF = S::LDS_FLOATS, OFF_REL = OFF + 12 * RLD, LDS_FLOATS = OFF_REL + 16;
    int n = 0;  // steps
    struct Out {
        float *lds;
        int n;
        const RowsRel &row;
        template <int LPR, int NV> __device__ __forceinline__ void store(const floatx4 (&rv)[4][NV], int lane) const {
            int64_t u[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) u[p] = row.rel[p] < 0 ? -1 : p;
            store_rows<LPR>(rv, lds + (n < 3 ? OFF + 4 * n * RLD : S::FREE), RLD, u, lane);
            const int lo = lane & 1 ? row.rel[1] : row.rel[0], hi = lane & 1 ? row.rel[3] : row.rel[2];
            if (lane < 4) ((int32_t *)lds)[OFF_REL + 4 * n + lane] = lane & 2 ? hi : lo;
        }
    };
    __device__ __forceinline__ Out out(float *lds, const RowsRel &row) { return {lds, n++, row}; }
    __device__ __forceinline__ void flush(const float *lds, const XTable &x) {
        using M = XMatrix<D, true>;
        constexpr int NK = M::NK;
        const int lane = opaque_tid(), a = lane & 15, q = lane >> 4;
        const float *src = lds + (a < 12 ? OFF + a * RLD : S::FREE + (a - 12) * RLD) + 8 * q;  // whatever lies there, beyond the last step
        const int32_t rel = ((const int32_t *)lds)[OFF_REL + a];
        const bool have = a < 4 * n && rel >= 0;
        n = 0;
        uint16_t *dst = x.X + (int64_t)rel * x.ldx + 8 * q;
        x_rows_from_memory<D, true>(opaque(x.mat), lane, [&](bf16x8 (&xp)[2][NK]) {
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
                bf16x8 part[2];
                M::cut(*(const float4 *)(src + 32 * kb), *(const float4 *)(src + 32 * kb + 4), part);
                xp[0][kb] = part[0];
                xp[1][kb] = part[1];
            }
        }, [&](int P, const floatx4 (&v)[2]) {
            if (have) store_x8<true>(dst + 32 * P, v);
        });
    }
};

// One step by itself.
template <class S>
__device__ __forceinline__ void single_step(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                            const float *__restrict__ values, const void *__restrict__ Z, float *__restrict__ R,
                                            int64_t ldr, int64_t r0, const int32_t *__restrict__ list, int count,
                                            int32_t *__restrict__ err_flag, int blk, float *lds) {
    S::init(lds, opaque_tid());
    const RowsRel rel = rows_rel(list, count, blk);
    const RowsDesc d = rows_desc(rel, rows_bounds(indptr, r0, rel), count, blk);
    int32_t idv[S::NIDS];
    S::ids(indices, d, opaque_tid(), idv);
    wait_ids(idv);
    S::solve(values, Z, err_flag, lds, d, idv, [] {}, [] {}, [] {}, RowsOut{R + r0 * ldr, ldr, d.row});
}

// The whole list, for any grid that is a multiple of eight: each die takes a contiguous eighth of the steps (see xcd_step), its
// wavefronts in turn.  List entry, row descriptor, column id and table row are four dependent loads; while a step is solved the
// first three of the wavefront's next step are on their way, so that only the last is waited for.
// store(lds, desc.row) gives the `out` of a step, done(lds, last) is called after it.
template <class S, class Store, class Done>
__device__ __forceinline__ void walk_steps(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                           const float *__restrict__ values, const void *__restrict__ Z, int64_t r0,
                                           const int32_t *__restrict__ list, int count, int32_t *__restrict__ err_flag, float *lds,
                                           Store &&store, Done &&done) {
    const WalkRange range = walk_range(blockIdx.x, gridDim.x, count);
    const int end = range.end, stride = range.stride;
    int blk = range.blk;
    if (blk >= end) return;
    S::init(lds, opaque_tid());
    auto clamp = [&](int b) { return b < end ? b : end - 1; };  // beyond the end: the last step again, unused
    RowsRel rel = rows_rel(list, count, blk), rel2;
    RowsDesc d = rows_desc(rel, rows_bounds(indptr, r0, rel), count, blk), dn;
    int32_t idv[S::NIDS], idn[S::NIDS];
    S::ids(indices, d, opaque_tid(), idv);
    rel = rows_rel(list, count, clamp(blk + stride));
    wait_ids(idv);
    for (;;) {
        const int next = blk + stride;
        RowsBounds w;
        float *here = opaque(lds);
        S::solve(
            opaque(values), opaque(Z), err_flag, here, d, idv,
            [&] {
                w = rows_bounds(opaque(indptr), r0, rel);
                rel2 = rows_rel(opaque(list), count, clamp(next + stride));
            },
            [&] {
                dn = rows_desc(rel, w, count, clamp(next));
                S::ids(opaque(indices), dn, opaque_tid(), idn);
            },
            [&] { wait_ids(idn); }, store(here, d.row));
        done(here, next >= end);
        if (next >= end) break;
        wave_sync();  // the next step reuses the LDS buffers
        blk = next;
        d = dn;
        rel = rel2;
#pragma unroll
        for (int n = 0; n < S::NIDS; ++n) idv[n] = idn[n];
    }
}
template <class S>
__device__ __forceinline__ void walk_steps(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                           const float *__restrict__ values, const void *__restrict__ Z, float *__restrict__ R,
                                           int64_t ldr, int64_t r0, const int32_t *__restrict__ list, int count,
                                           int32_t *__restrict__ err_flag, float *lds) {
    R += r0 * ldr;
    walk_steps<S>(indptr, indices, values, Z, r0, list, count, err_flag, lds,
                  [&](float *, const RowsRel &row) { return RowsOut{opaque(R), opaque(ldr), row}; }, [](float *, bool) {});
}
template <class S, int D>
__device__ __forceinline__ void walk_steps_x(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                             const float *__restrict__ values, const void *__restrict__ Z, XTable x, int64_t r0,
                                             const int32_t *__restrict__ list, int count, int32_t *__restrict__ err_flag, float *lds) {
    Parked<S, D> parked;
    x.X += r0 * x.ldx;
    walk_steps<S>(indptr, indices, values, Z, r0, list, count, err_flag, lds,
                  [&](float *here, const RowsRel &row) { return parked.out(here, row); },
                  [&](float *here, bool last) {
                      if (parked.n < 4 && !last) return;
                      wave_sync();
                      parked.flush(here, x);
                  });
}

// Wavefronts of 64 threads and `lds_bytes` that the device holds at a time (the runtime is asked once per kernel and process).
template <class K> inline int resident_waves(K *kernel, size_t lds_bytes, int num_cu) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)kernel, 64, lds_bytes) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        n = 8;
    }
    return n * num_cu;
}

// What a launch of walk_steps knows about its list: the steps it can hold at most, and those that an earlier call saw (or -1).
struct WalkSize {
    int num_cu;
    int64_t capacity, hint;
};

}  // namespace als
