// Walking the list of a row class that is worked four rows per step and wavefront.
#pragma once

#include "dual_common.h"

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
//   solve(values, Z, R, ldr, err_flag, lds, desc, idv, loaded, between, last)
//         one step; R is row r0 of the output; calls `loaded` when the loads of the entries are under way, `between` once the
//         entries have been used for S, before the elimination, and `last` before the stores.

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
    S::solve(values, Z, R + r0 * ldr, ldr, err_flag, lds, d, idv, [] {}, [] {}, [] {});
}

// The whole list, for any grid that is a multiple of eight: each die takes a contiguous eighth of the steps (see xcd_step), its
// wavefronts in turn.  List entry, row descriptor, column id and table row are four dependent loads; while a step is solved the
// first three of the wavefront's next step are on their way, so that only the last is waited for.
template <class S>
__device__ __forceinline__ void walk_steps(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                           const float *__restrict__ values, const void *__restrict__ Z, float *__restrict__ R,
                                           int64_t ldr, int64_t r0, const int32_t *__restrict__ list, int count,
                                           int32_t *__restrict__ err_flag, float *lds) {
    const WalkRange range = walk_range(blockIdx.x, gridDim.x, count);
    const int end = range.end, stride = range.stride;
    int blk = range.blk;
    if (blk >= end) return;
    S::init(lds, opaque_tid());
    R += r0 * ldr;
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
        S::solve(
            opaque(values), opaque(Z), opaque(R), opaque(ldr), err_flag, opaque(lds), d, idv,
            [&] {
                w = rows_bounds(opaque(indptr), r0, rel);
                rel2 = rows_rel(opaque(list), count, clamp(next + stride));
            },
            [&] {
                dn = rows_desc(rel, w, count, clamp(next));
                S::ids(opaque(indices), dn, opaque_tid(), idn);
            },
            [&] { wait_ids(idn); });
        if (next >= end) break;
        wave_sync();  // the next step reuses the LDS buffers
        blk = next;
        d = dn;
        rel = rel2;
#pragma unroll
        for (int n = 0; n < S::NIDS; ++n) idv[n] = idn[n];
    }
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
