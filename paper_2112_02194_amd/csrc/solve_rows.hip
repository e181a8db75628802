// als_solve_rows orchestration: classify the rows of the requested range by their number of
// stored entries, then run the kernels each class needs (paper Algorithm 1 lines 3-10; long rows
// are cut into segments in the spirit of Section 4.3).  Nothing here waits for the GPU: the class
// counts stay in device memory, every row kernel reads the length of its list there and covers the
// list whatever its grid, and grids are sized from the counts of the previous call on the same
// matrix when there was one (a hint: a wrong or missing hint costs speed, never correctness).
#include <type_traits>

#include "als_internal.h"
#include "factor.h"

namespace als {

als_status launch_primal(als_ctx *ctx, const als_csr *Y, const als_table *V, const float *G, const als_params *prm, als_table *X,
                         int64_t r0, const LongRow *long_rows, const Segment *segs, const int32_t *counters, int64_t seg_capacity,
                         StepGrid g_long, StepGrid g_seg, const int32_t *row_list, const int32_t *row_count, StepGrid g_row, hipStream_t s);
als_status launch_dual_prepare(als_ctx *ctx, const als_table *V, const float *G, const als_params *prm,
                               const als_csr *entries, int64_t r0, int64_t r1, bool factored, hipStream_t s);
als_status launch_dual_rows(als_ctx *ctx, const als_csr *Y, als_table *X, int64_t r0, int64_t r1, int dual_max,
                            const als_params *prm, const int32_t *const lists[10], const int32_t *const counts_dev[10],
                            const int64_t caps[10], const int hints[10], hipStream_t s);
als_status launch_cg_free(als_ctx *ctx, const als_csr *Y, const als_table *V, const float *G, const als_params *prm,
                          als_table *X, int64_t r0, const int32_t *const lists[10], const int32_t *const counts_dev[10],
                          const int64_t caps[10], const int hints[10], hipStream_t s);
int dual_supported_max_k(int d);

constexpr int DEFAULT_SPLIT = 512;
constexpr int SEG_CAPACITY = 32768;  // segments whose partial statistics the workspace holds ((d*d + d) floats each)
constexpr int MAX_SEGS_PER_ROW = 128;
constexpr int64_t BLIND_PRIMAL = 1 << 20;  // see step_grid; workgroups of up to four wavefronts

__global__ void clear_counters_kernel(int32_t *counters, long long *long_stat, int32_t *queue) {
    const int t = threadIdx.x;
    if (t < 2 * QUEUE_PARTS) queue[t * QUEUE_STRIDE] = 0;
    if (t < 16 && t != 2 && t != 4) counters[t] = 0;  // [2] is the sticky error flag, [4] the CSR check flag
    if (t < 2) long_stat[t] = 0;
}

constexpr int CLS_THREADS = 256;
// Rows per thread: eight, so that few workgroups reserve places with atomics, but two while each of those workgroups has a
// compute unit to itself, where the rounds of a thread, one after the other, are what is waited for.  Epoch of 50k x 30k, eight / two:
// 325 / 312 us; the kernel for 2 x 1M rows 35 / 59 us, for 2 x 10M rows 191 / 465 us.
constexpr int CLS_RPT_MANY = 8, CLS_RPT_FEW = 2;
// Up to this many rows one large workgroup does what takes four dependent launches otherwise (clearing, the long rows' sums, the
// lists, their lengths for the host).  Epoch of 2000 x 1500 113 -> 95 us, 256 folded-in rows (d = 128) 85.7 -> 80.4 us; eight
// rows a thread are all it can hold in registers.  At the line, 8192 rows of 12 entries / without entries, one launch against
// four with two rows a thread: d = 16 35 / 31 against 38 / 38 us a call, d = 128 101 / 89 against 100 / 93 us.
constexpr int CLS_ONE_THREADS = 1024, CLS_ONE_RPT = 8, CLS_ONE_ROWS = CLS_ONE_THREADS * CLS_ONE_RPT;
struct ListOffsets { int64_t v[11]; };  // start of each dual class list (and the end of the last), passed by value

// Entries and rows beyond the requested split threshold, summed per workgroup and added with one atomic
// each (integer sums: the order does not matter).
template <int RPT>
__global__ __launch_bounds__(CLS_THREADS) void long_stat_kernel(const int64_t *__restrict__ indptr, int64_t r0,
                                                               int64_t r1, int64_t split,
                                                               unsigned long long *__restrict__ long_stat) {
    __shared__ unsigned long long red[2][CLS_THREADS / 64];
    unsigned long long ent = 0, cnt = 0;
    const int64_t u0 = r0 + (int64_t)blockIdx.x * (CLS_THREADS * RPT);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int64_t u = u0 + (int64_t)i * CLS_THREADS + threadIdx.x;
        if (u < r1) {
            const int64_t k = indptr[u + 1] - indptr[u];
            if (k > split) {
                ent += (unsigned long long)k;
                cnt += 1;
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        ent += __shfl_xor(ent, off);
        cnt += __shfl_xor(cnt, off);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wave] = ent;
        red[1][wave] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long e = 0, c = 0;
        for (int w = 0; w < CLS_THREADS / 64; ++w) {
            e += red[0][w];
            c += red[1][w];
        }
        if (c) {
            atomicAdd(&long_stat[0], e);
            atomicAdd(&long_stat[1], c);
        }
    }
}

// The split threshold in use: the requested one, raised until the segments of all long rows fit the
// workspace.  With s >= entries_beyond / (SEG_CAPACITY / 2) the rows longer than s number at most
// SEG_CAPACITY / 2 and their segments (each row: at most k/s + 1) at most SEG_CAPACITY.
__device__ __forceinline__ int32_t decide_split(const unsigned long long *__restrict__ long_stat, int64_t split) {
    const unsigned long long need = (long_stat[0] + SEG_CAPACITY / 2 - 1) / (SEG_CAPACITY / 2);
    unsigned long long s = (unsigned long long)split;
    if (need > s) s = need;
    return (int32_t)(s > 0x7fffffffull ? 0x7fffffffull : s);
}

// 0 = mid list, 1..8 = dual classes by ceil(k/16), 9 = k <= 4, 10 = 5 <= k <= 8
__device__ __forceinline__ int row_class(int64_t k, int64_t dual_max) {
    return k > dual_max ? 0 : (k <= 4 ? 9 : (k <= 8 ? 10 : (int)((k + 15) / 16)));
}
// where the length of list `cls` stands among the counters
__device__ __forceinline__ int class_counter(int cls) { return cls == 0 ? 3 : (cls <= 8 ? 8 + cls - 1 : cls - 4); }

// a / b rounded up, for 0 < a and 0 < b < 2^31 (a 64-bit division takes about five times the instructions of a 32-bit one)
__device__ __forceinline__ int64_t divide_up(int64_t a, int64_t b) {
    return a <= 0x7fffffff ? (int64_t)(((uint32_t)a + (uint32_t)b - 1u) / (uint32_t)b) : (a + b - 1) / b;
}
__device__ __forceinline__ int segments_of(int64_t k, int64_t split) {
    const int64_t nseg = divide_up(k, split);
    return (int)(nseg < MAX_SEGS_PER_ROW ? nseg : MAX_SEGS_PER_ROW);
}
// Row u with k > split entries from b on becomes long row `slot` with its balanced segments from `first` on; false where they
// do not fit.
__device__ __forceinline__ bool put_long_row(int64_t u, int64_t b, int64_t k, int64_t split, int slot, int first,
                                             LongRow *__restrict__ long_rows, Segment *__restrict__ segs) {
    const int nseg = segments_of(k, split);
    const int64_t len = divide_up(k, nseg), e = b + k;
    if (slot >= SEG_CAPACITY / 2 || first + nseg > SEG_CAPACITY) return false;
    long_rows[slot].row = u;
    long_rows[slot].seg_first = first;
    long_rows[slot].nseg = nseg;
    for (int g = 0; g < nseg; ++g) {
        const int64_t start = b + g * len, stop = b + (g + 1) * len;
        segs[first + g].begin = start < e ? start : e;
        segs[first + g].end = stop < e ? stop : e;
    }
    return true;
}

// One workgroup per CLS_THREADS * RPT consecutive rows of [r0, r1):
//   k = 0               X[u] = 0
//   0 < k <= dual_max   appended to the dual list of its class: k <= 4, 5..8, else ceil(k/16) in 1..8
//                       (row id relative to r0)
//   dual_max < k <= split  appended to the mid list (primal, one workgroup per row)
//   k > split           becomes a long row cut into balanced segments of about `split` entries
//                       (at most MAX_SEGS_PER_ROW of them); split is the threshold of decide_split, left in
//                       counters[7] too
// Positions are reserved with one atomic per workgroup and list (counts gathered in LDS; with two per long row, whose answers a
// wavefront waited for up to eight times, the 1M rows of a heavy-tailed half took 74 us instead of 17).  Rows keep
// their order inside a wavefront's 64; the wavefronts of a workgroup, and the workgroups, come in any order, which can change from call to
// call.  No result depends on it, and neighbouring rows still stand near each other.  A matrix whose indptr does not fit its nnz can ask
// for more long rows or segments than the workspace holds; those rows are dropped and the error flag is set.  So are, when Z
// holds one row per entry (entry_limit = nnz, else INT64_MAX), rows with entries outside those that Gather walks, from
// indptr[r0] to indptr[r1] and below entry_limit: an indptr that is not monotone has such rows, and Z has nothing for them.
template <bool BF16, int RPT>
__global__ __launch_bounds__(CLS_THREADS) void classify_kernel(
    const int64_t *__restrict__ indptr, int64_t r0, int64_t r1, int64_t dual_max, int d,
    void *__restrict__ X, int64_t ldx, int32_t *__restrict__ counters, LongRow *__restrict__ long_rows,
    Segment *__restrict__ segs, int32_t *__restrict__ mid_list, int64_t cap_mid, int32_t *__restrict__ dual_lists,
    ListOffsets list_off, int64_t entry_limit, const unsigned long long *__restrict__ long_stat, int64_t split_wanted) {
    __shared__ int32_t cnt[13], base[13];  // lists 0..10, long rows, their segments
    const int t = threadIdx.x;
    if (t < 13) cnt[t] = 0;
    __syncthreads();
    const int64_t split = decide_split(long_stat, split_wanted);
    if (blockIdx.x == 0 && t == 0) counters[7] = (int32_t)split;
    const bool by_entry = entry_limit != INT64_MAX;
    const int64_t first_entry = by_entry && indptr[r0] > 0 ? indptr[r0] : 0;
    const int64_t end_entry = by_entry && indptr[r1] < entry_limit ? indptr[r1] : entry_limit;
    const int64_t u0 = r0 + (int64_t)blockIdx.x * (CLS_THREADS * RPT);
    int cls[RPT], pos[RPT], seg[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int64_t u = u0 + (int64_t)i * CLS_THREADS + t;  // coalesced indptr reads
        cls[i] = -1;
        pos[i] = seg[i] = 0;
        if (u < r1) {
            const int64_t b = indptr[u], e = indptr[u + 1], k = e - b;
            if (b < first_entry || e > end_entry) {
                atomicOr(&counters[2], 2);
            } else if (k <= 0) {
                for (int c = 0; c < d; ++c) store_elem<BF16>(X, u * ldx + c, 0.f);
            } else if (k > split) {
                cls[i] = 11;
                pos[i] = atomicAdd(&cnt[11], 1);
                seg[i] = atomicAdd(&cnt[12], segments_of(k, split));
            } else {
                cls[i] = row_class(k, dual_max);
                pos[i] = atomicAdd(&cnt[cls[i]], 1);
            }
        }
    }
    __syncthreads();
    if (t < 13 && cnt[t] > 0) base[t] = atomicAdd(&counters[t < 11 ? class_counter(t) : t - 11], cnt[t]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        if (cls[i] < 0) continue;
        if (cls[i] == 11) {
            const int64_t u = u0 + (int64_t)i * CLS_THREADS + t, b = indptr[u];
            if (!put_long_row(u, b, indptr[u + 1] - b, split, base[11] + pos[i], base[12] + seg[i], long_rows, segs)) atomicOr(&counters[2], 2);
            continue;
        }
        const int32_t rel = (int32_t)(u0 + (int64_t)i * CLS_THREADS + t - r0);
        const int64_t at = (int64_t)base[cls[i]] + pos[i];
        if (cls[i] == 0) {
            if (at < cap_mid) mid_list[at] = rel;
            else atomicOr(&counters[2], 2);
        } else {
            const int c = cls[i] - 1;  // class ids 1..10 -> lists 0..9
            if (at < list_off.v[c + 1] - list_off.v[c]) dual_lists[list_off.v[c] + at] = rel;
            else atomicOr(&counters[2], 2);
        }
    }
}

// Clamp the counts to what was stored (only a matrix inconsistent with its nnz exceeds a capacity) and copy
// them into the host-visible hint slot, sequence number last.
__global__ void publish_counts_kernel(int32_t *__restrict__ counters, int64_t cap_mid, ListOffsets list_off,
                                      int32_t *__restrict__ hint, uint32_t seq) {
    const int t = threadIdx.x;
    if (t == 0) {
        if (counters[2] & 2) {  // something was dropped: no long rows at all rather than half-written ones
            counters[0] = 0;
            counters[1] = 0;
        }
        if (counters[3] > cap_mid) counters[3] = (int32_t)cap_mid;
        for (int c = 0; c < 10; ++c) {
            const int ci = c < 8 ? 8 + c : c - 3;
            const int64_t cap = list_off.v[c + 1] - list_off.v[c];
            if (counters[ci] > cap) counters[ci] = (int32_t)cap;
        }
    }
    __syncthreads();
    if (t < 16) hint[t] = counters[t];
    __threadfence_system();
    __syncthreads();
    if (t == 0) {
        ((volatile int32_t *)hint)[16] = (int32_t)seq;
        __threadfence_system();
    }
}

// The rows u0 + j of X with bit j of the wavefront-uniform `which` become zero, 16 bytes a lane, as many rows at a time as the
// wavefront spans.  (With one thread per row, one element after the other, as in classify_kernel, a call with 8192 empty rows took 574 us
// for d = 128, fp32, and 75 us for d = 16: all of them wait for one compute unit.  So it takes 89 and 31 us.)
template <bool BF16> __device__ __forceinline__ void zero_rows(void *X, int64_t ldx, int d, int64_t u0, unsigned long long which) {
    constexpr int ES = BF16 ? 2 : 4;
    const int lane = threadIdx.x & 63, shift = __ffs(d * ES / 16) - 1;  // 2, 4, .. 32 lanes per row
    const int64_t mine = lane >> shift;
    for (int j = 0; which && j < 64; j += 64 >> shift) {
        if (which >> (j + mine) & 1)
            *(float4 *)((char *)X + (u0 + j + mine) * ldx * ES + 16 * (lane & ((1 << shift) - 1))) = make_float4(0.f, 0.f, 0.f, 0.f);  // (rows are 16-byte aligned)
    }
}

// The four kernels above in one, for at most CLS_ONE_ROWS rows: one workgroup, everything counted in LDS.  The same lists,
// segments, counters and hint.
struct SortArgs {
    const int64_t *indptr;
    int64_t r0, r1, dual_max;
    int d;
    void *X;
    int64_t ldx;
    int32_t *counters;
    LongRow *long_rows;
    Segment *segs;
    int32_t *mid_list;
    int64_t cap_mid;
    int32_t *dual_lists;
    ListOffsets list_off;
    int64_t entry_limit, split_wanted;
    int32_t *hint;
    uint32_t seq;
    int32_t *queue;
};
template <bool BF16> __device__ __forceinline__ void classify_one(const SortArgs &a) {
    const int64_t *__restrict__ indptr = a.indptr;
    const int64_t r0 = a.r0, r1 = a.r1, dual_max = a.dual_max, ldx = a.ldx, cap_mid = a.cap_mid, entry_limit = a.entry_limit, split_wanted = a.split_wanted;
    const int d = a.d;
    void *__restrict__ X = a.X;
    int32_t *__restrict__ counters = a.counters, *__restrict__ mid_list = a.mid_list, *__restrict__ dual_lists = a.dual_lists, *__restrict__ hint = a.hint,
                          *__restrict__ queue = a.queue;
    LongRow *__restrict__ long_rows = a.long_rows;
    Segment *__restrict__ segs = a.segs;
    const ListOffsets &list_off = a.list_off;
    const uint32_t seq = a.seq;
    __shared__ int32_t n[16];  // as in `counters`; [2]: flag bits set here
    __shared__ unsigned long long long_stat[1];  // entries of the rows beyond the requested split
    const int t = threadIdx.x;
    if (t < 16) n[t] = 0;
    if (t < 2 * QUEUE_PARTS) queue[t * QUEUE_STRIDE] = 0;
    if (t == 0) long_stat[0] = 0;
    const bool by_entry = entry_limit != INT64_MAX;
    const int64_t first_entry = by_entry && indptr[r0] > 0 ? indptr[r0] : 0;
    const int64_t end_entry = by_entry && indptr[r1] < entry_limit ? indptr[r1] : entry_limit;
    int64_t b[CLS_ONE_RPT], e[CLS_ONE_RPT];
#pragma unroll
    for (int i = 0; i < CLS_ONE_RPT; ++i) {
        const int64_t u = r0 + (int64_t)i * CLS_ONE_THREADS + t;
        b[i] = e[i] = 0;
        if (u < r1) {
            b[i] = indptr[u];
            e[i] = indptr[u + 1];
        }
    }
    __syncthreads();
    unsigned long long beyond = 0;
#pragma unroll
    for (int i = 0; i < CLS_ONE_RPT; ++i) beyond += e[i] - b[i] > split_wanted ? (unsigned long long)(e[i] - b[i]) : 0ull;
    // Sums in one place of LDS go there lane by lane: with an address that is known to be the same in all lanes, the compiler adds up the
    // wavefront's values first, in a loop over its lanes that takes a microsecond.
    int here = 0;
    asm volatile("" : "+v"(here));
    if (beyond) atomicAdd(&long_stat[here], beyond);
    __syncthreads();
    const int64_t split = decide_split(long_stat, split_wanted);
    unsigned empty = 0, longs = 0;  // bit i: this thread's row i
    int nsegs = 0;                  // segments of its long rows
#pragma unroll
    for (int i = 0; i < CLS_ONE_RPT; ++i) {
        const int64_t u = r0 + (int64_t)i * CLS_ONE_THREADS + t, k = e[i] - b[i];
        if (u >= r1) continue;
        if (b[i] < first_entry || e[i] > end_entry) {
            atomicOr(&n[2], 2);
        } else if (k <= 0) {
            empty |= 1u << i;
        } else if (k > split) {
            longs |= 1u << i;
            nsegs += segments_of(k, split);
        } else {
            const int c = row_class(k, dual_max);
            const int64_t at = atomicAdd(&n[class_counter(c)], 1);
            const int64_t cap = c == 0 ? cap_mid : list_off.v[c] - list_off.v[c - 1];
            if (at < cap) (c == 0 ? mid_list : dual_lists + list_off.v[c - 1])[at] = (int32_t)(u - r0);
            else atomicOr(&n[2], 2);
        }
    }
    // what most calls have few of, in a loop of its own (unrolled with the rest it would cost the kernel its registers)
    int slot = 0, first = 0;
    if (longs) {
        slot = atomicAdd(&n[here], __popc(longs));
        first = atomicAdd(&n[here + 1], nsegs);
    }
#pragma unroll 1
    for (int i = 0; __any((longs | empty) >> i); ++i) {
        const int64_t u = r0 + (int64_t)i * CLS_ONE_THREADS + t;
        if (longs >> i & 1) {
            int64_t from = b[0], to = e[0];  // of row i, without waiting for indptr again
#pragma unroll
            for (int j = 1; j < CLS_ONE_RPT; ++j) {
                from = i == j ? b[j] : from;
                to = i == j ? e[j] : to;
            }
            const int64_t k = to - from;
            if (!put_long_row(u, from, k, split, slot, first, long_rows, segs)) atomicOr(&n[2], 2);
            ++slot;
            first += segments_of(k, split);
        }
        zero_rows<BF16>(X, ldx, d, u - (t & 63), __ballot(empty >> i & 1));
    }
    __syncthreads();
    if (t < 16 && t != 4) {  // [4] is the CSR check flag
        const int32_t flag = counters[2] | n[2];  // the error flag is sticky
        int32_t v = n[t];
        if (t == 2) v = flag;
        if (t == 7) v = (int32_t)split;
        if (t < 2 && (flag & 2)) v = 0;  // something was dropped: no long rows at all rather than half-written ones
        if (t == 3 && v > cap_mid) v = (int32_t)cap_mid;
        const int c = t >= 8 ? t - 8 : t + 3;  // list whose length stands here
        if (t == 5 || t == 6 || t >= 8) {
            const int64_t cap = list_off.v[c + 1] - list_off.v[c];
            if (v > cap) v = (int32_t)cap;
        }
        if (t != 2) counters[t] = v;
        else if (n[2]) atomicOr(&counters[2], n[2]);  // the factorisation beside it may be setting its bit
        hint[t] = v;
    }
    if (t < 64) __threadfence_system();
    if (t == 0) {
        ((volatile int32_t *)hint)[16] = (int32_t)seq;
        __threadfence_system();
    }
}

template <bool BF16> __global__ __launch_bounds__(CLS_ONE_THREADS) void classify_one_kernel(SortArgs a) { classify_one<BF16>(a); }

// With the shared factor of the dual rows in a second workgroup: neither needs the other.  Epoch of 2000 x 1500 (d = 16)
// 90 -> 82 us, 256 rows folded in (d = 128) 80.8 -> 75.2, 3000 rows (d = 64, bf16) 59 -> 53 us; on their own the two take 4 to 6 us and
// 3 (d = 16) to 31 us (d = 128).
template <int D, bool BF16>
__global__ __launch_bounds__(CLS_ONE_THREADS) void sort_factor_kernel(SortArgs a, const float *__restrict__ G, float alpha, float lambda,
                                                                     float *__restrict__ Linv, float *__restrict__ LinvT) {
    extern __shared__ double fa[];
    if (blockIdx.x == 0) classify_one<BF16>(a);
    else if (threadIdx.x < FACTOR_THREADS) factor<D>(G, alpha, lambda, Linv, LinvT, a.counters + 2, fa);  // (the other wavefronts end: no barrier waits for them)
}

template <int D, bool BF16>
static als_status launch_sort_factor(als_ctx *ctx, const SortArgs &a, const float *G, const als_params *prm, hipStream_t s) {
    constexpr int lds_bytes = (int)FactorCfg<D>::LDS_BYTES;
    static const hipError_t attr = hipFuncSetAttribute((const void *)sort_factor_kernel<D, BF16>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);  // once per process
    ALS_HIP(ctx, attr);
    float *Linv = (float *)((char *)ctx->small.p + SM_FACTOR);
    hipLaunchKernelGGL((sort_factor_kernel<D, BF16>), dim3(2), dim3(CLS_ONE_THREADS), lds_bytes, s, a, G, prm->alpha, prm->lambda, Linv,
                       Linv + 128 * 128);
    return ALS_OK;
}

als_status launch_solve_rows(als_ctx *ctx, const als_csr *Y, const als_table *V, const float *G,
                             const als_params *prm_in, als_table *X, int64_t r0, int64_t r1, hipStream_t s) {
    // ALS_SOLVER_CG_FREE: the rows of the class lists never see an assembled system; longer rows take
    // conjugate gradients on their assembled one
    const bool cg_free = prm_in->solver == ALS_SOLVER_CG_FREE;
    als_params prm_rows = *prm_in;
    if (cg_free) prm_rows.solver = ALS_SOLVER_CG;
    const als_params *prm = &prm_rows;
    const int64_t nrows = r1 - r0;
    if (nrows > INT32_MAX) return fail(ctx, ALS_EINVAL, "row range longer than 2^31-1: call per sub-range");
    const int64_t split = prm->split_nnz > 0 ? prm->split_nnz : DEFAULT_SPLIT;
    int dual_max = 0;
    if (prm->path != ALS_PATH_PRIMAL) {
        dual_max = dual_supported_max_k(V->d);
        if (prm->dual_max_k > 0 && prm->dual_max_k < dual_max) dual_max = prm->dual_max_k;
        if (dual_max > split) dual_max = (int)split;
        // conjugate gradients on the k x k systems run in the one-row-per-wavefront kernels, which exist for d >= 64
        if (prm_in->solver == ALS_SOLVER_CG && V->d < 64) dual_max = 0;
    }
    // list capacities: class c (k > 16(c-1)) holds at most nnz/(16(c-1)+1) rows, the mid list at most
    // nnz/(dual_max+1)
    int64_t off[11];  // lists 0..7: classes by ceil(k/16); list 8: k <= 4; list 9: 5 <= k <= 8
    off[0] = 0;
    for (int c = 1; c <= 10; ++c) {
        int64_t cap = 0;
        if (c <= 8) {
            if (dual_max > 16 * (c - 1)) cap = std::min<int64_t>(nrows, Y->nnz / (16 * (c - 1) + 1) + 1);
        } else if (dual_max > 0) {
            cap = std::min<int64_t>(nrows, Y->nnz / (c == 9 ? 1 : 5) + 1);
        }
        off[c] = off[c - 1] + cap;
    }
    const int64_t cap_mid = std::min<int64_t>(nrows, Y->nnz / (dual_max + 1) + 1);
    const size_t off_seg = (size_t)(SEG_CAPACITY / 2) * sizeof(LongRow);
    const size_t off_lists = off_seg + (size_t)SEG_CAPACITY * sizeof(Segment);
    // + 16 bytes: the row kernels read a wavefront's four list entries with one 16-byte load
    als_status st = ensure(ctx, ctx->lists, off_lists + (size_t)(cap_mid + off[10]) * sizeof(int32_t) + 16);
    if (st != ALS_OK) return st;
    LongRow *long_rows = (LongRow *)ctx->lists.p;
    Segment *segs = (Segment *)((char *)ctx->lists.p + off_seg);
    int32_t *mid_list = (int32_t *)((char *)ctx->lists.p + off_lists);
    int32_t *dual_lists = mid_list + cap_mid;
    int32_t *counters = (int32_t *)((char *)ctx->small.p + SM_COUNTERS);
    unsigned long long *long_stat = (unsigned long long *)((char *)ctx->small.p + SM_LONGSTAT);
    int32_t *queue = (int32_t *)((char *)ctx->small.p + SM_QUEUE);
    ListOffsets list_off;
    for (int c = 0; c <= 10; ++c) list_off.v[c] = off[c];

    // ---- hint slot of this (matrix, range, class shape): counts of the previous such call, if they have arrived
    int slot = -1, lru = 0;
    for (int i = 0; i < N_HINTS; ++i) {
        const HintSlot &h = ctx->hints[i];
        if (h.seq != 0 && h.indptr == (const void *)Y->indptr && h.rows == Y->rows && h.nnz == Y->nnz && h.r0 == r0 &&
            h.r1 == r1 && h.split == (int32_t)split && h.dual_max == dual_max && h.d == V->d)
            slot = i;
        if (ctx->hints[i].seq < ctx->hints[lru].seq) lru = i;
    }
    int hint[16];
    for (int i = 0; i < 16; ++i) hint[i] = -1;
    if (++ctx->hint_seq == 0) ctx->hint_seq = 1;
    if (slot >= 0) {
        // whatever call with this key the GPU has finished last left its counts here (the host may be several
        // calls ahead of the GPU: the hint need not come from the call just before this one)
        const volatile int32_t *hc = ctx->hint_counts + (size_t)slot * HINT_INTS;
        const uint32_t stamp = (uint32_t)hc[16];
        if (stamp != 0 && stamp - ctx->hints[slot].first_seq < 0x80000000u)
            for (int i = 0; i < 16; ++i) hint[i] = hc[i];
    } else {
        slot = lru;
        ctx->hints[slot].first_seq = ctx->hint_seq;
    }
    HintSlot &hs = ctx->hints[slot];
    hs.indptr = Y->indptr; hs.rows = Y->rows; hs.nnz = Y->nnz; hs.r0 = r0; hs.r1 = r1;
    hs.split = (int32_t)split; hs.dual_max = dual_max; hs.d = V->d;
    hs.seq = ctx->hint_seq;

    // Fewer entries than table rows: only the rows that the entries name are transformed, in the order of the entries, and
    // the row kernels find entry p at row p of Z.  Measured against the whole table of 1M rows (d = 128, fp32 / bf16), us:
    // 3 900 entries 440 -> 171 / 294 -> 148, 0.45M entries 585 -> 459 / 405 -> 300, 0.9M entries 661 -> 655 / 454 -> 450.
    const bool by_entry = dual_max > 0 && !cg_free && Y->nnz <= INT32_MAX && Y->nnz < V->rows;
    als_csr by_position = *Y;

    timer_begin(ctx, T_CLASSIFY, s);
    const bool bf = V->dtype == ALS_BF16;
    const int64_t entry_limit = by_entry ? Y->nnz : INT64_MAX;
    int32_t *hint_out = ctx->hint_counts_dev + (size_t)slot * HINT_INTS;
    bool factored = false;
    if (nrows <= CLS_ONE_ROWS) {
        const SortArgs a = {Y->indptr, r0, r1, (int64_t)dual_max, V->d, X->data, X->ld, counters, long_rows, segs, mid_list, cap_mid, dual_lists,
                            list_off, entry_limit, split, hint_out, hs.seq, queue};
        factored = dual_max > 0 && !cg_free;
        if (!factored) {
            hipLaunchKernelGGL(bf ? classify_one_kernel<true> : classify_one_kernel<false>, dim3(1), dim3(CLS_ONE_THREADS), 0, s, a);
        } else {
#define ALS_SORT_CASE(dd) case dd: st = bf ? launch_sort_factor<dd, true>(ctx, a, G, prm, s) : launch_sort_factor<dd, false>(ctx, a, G, prm, s); break;
            switch (V->d) { ALS_SORT_CASE(16) ALS_SORT_CASE(32) ALS_SORT_CASE(64) ALS_SORT_CASE(128) }
#undef ALS_SORT_CASE
            if (st != ALS_OK) return st;
        }
    } else {
        hipLaunchKernelGGL(clear_counters_kernel, dim3(1), dim3(64), 0, s, counters, (long long *)long_stat, queue);
        auto sort = [&](auto rows_per_thread) {
            constexpr int RPT = decltype(rows_per_thread)::value;
            const unsigned cblocks = (unsigned)((nrows + CLS_THREADS * RPT - 1) / (CLS_THREADS * RPT));
            hipLaunchKernelGGL(long_stat_kernel<RPT>, dim3(cblocks), dim3(CLS_THREADS), 0, s, Y->indptr, r0, r1, split, long_stat);
            hipLaunchKernelGGL((bf ? classify_kernel<true, RPT> : classify_kernel<false, RPT>), dim3(cblocks), dim3(CLS_THREADS), 0,
                               s, Y->indptr, r0, r1, (int64_t)dual_max, V->d, X->data, X->ld, counters, long_rows, segs, mid_list,
                               cap_mid, dual_lists, list_off, entry_limit, (const unsigned long long *)long_stat, split);
        };
        if (nrows <= (int64_t)ctx->num_cu * CLS_THREADS * CLS_RPT_FEW) sort(std::integral_constant<int, CLS_RPT_FEW>{});
        else sort(std::integral_constant<int, CLS_RPT_MANY>{});
        hipLaunchKernelGGL(publish_counts_kernel, dim3(1), dim3(64), 0, s, counters, cap_mid, list_off, hint_out, hs.seq);
    }
    timer_end(ctx, s);
    ALS_HIP(ctx, hipGetLastError());

    if (by_entry) {
        if ((st = ensure(ctx, ctx->entry_ids, (size_t)std::max<int64_t>(Y->nnz, 1) * sizeof(int32_t))) != ALS_OK) return st;
        by_position.indices = (const int32_t *)ctx->entry_ids.p;
    }
    if (dual_max > 0 && !cg_free) {
        if ((st = launch_dual_prepare(ctx, V, G, prm, by_entry ? Y : nullptr, r0, r1, factored, s)) != ALS_OK) return st;
    }
    // segments: at most 2 nnz / split + 1 of them exist, and never more than the workspace holds
    const int64_t seg_capacity = std::min<int64_t>(SEG_CAPACITY, 2 * (Y->nnz / split) + 2);
    const int pt = primal_threads(V->d);
    const StepGrid g_long = step_grid(ctx->num_cu, pt, std::min<int64_t>(SEG_CAPACITY / 2, Y->nnz / split + 1), hint[0], 4, SEG_CAPACITY);
    const StepGrid g_seg = step_grid(ctx->num_cu, pt, seg_capacity, hint[1], 8, SEG_CAPACITY);
    const StepGrid g_row = step_grid(ctx->num_cu, pt, cap_mid, hint[3], 8, BLIND_PRIMAL, g_seg.known);  // one launch may take both
    if ((st = launch_primal(ctx, Y, V, G, prm, X, r0, long_rows, segs, counters, seg_capacity, g_long, g_seg, mid_list, counters + 3,
                            g_row, s)) != ALS_OK)
        return st;
    if (dual_max > 0) {
        const int32_t *lists[10], *counts_dev[10];
        int64_t caps[10];
        int hints[10];
        for (int c = 0; c < 10; ++c) {
            lists[c] = dual_lists + off[c];
            const int ci = c < 8 ? 8 + c : c - 3;  // counters [5], [6]: the two small classes
            counts_dev[c] = counters + ci;
            caps[c] = off[c + 1] - off[c];
            hints[c] = hint[ci];
        }
        st = cg_free ? launch_cg_free(ctx, Y, V, G, prm, X, r0, lists, counts_dev, caps, hints, s)
                     : launch_dual_rows(ctx, by_entry ? &by_position : Y, X, r0, r1, dual_max, prm, lists, counts_dev, caps, hints, s);
        if (st != ALS_OK) return st;
    }
    return ALS_OK;
}

// ---------------------------------------------------------------------------------------------- validation
__global__ __launch_bounds__(256) void check_csr_kernel(const int64_t *__restrict__ indptr,
                                                        const int32_t *__restrict__ indices, int64_t rows,
                                                        int64_t cols, int64_t nnz, int32_t *__restrict__ flag) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool bad = false;
    if (t == 0) bad = indptr[0] != 0 || indptr[rows] != nnz;
    for (int64_t u = t; u < rows; u += stride) bad |= indptr[u + 1] < indptr[u];
    for (int64_t p = t; p < nnz; p += stride) bad |= indices[p] < 0 || indices[p] >= cols;
    if (bad) atomicOr(flag, 1);
}

als_status launch_check_csr(als_ctx *ctx, const als_csr *Y, int32_t *flag_dev, hipStream_t s) {
    int64_t work = std::max<int64_t>(Y->rows, Y->nnz);
    unsigned blocks = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, (work + 255) / 256));
    hipLaunchKernelGGL(check_csr_kernel, dim3(blocks), dim3(256), 0, s, Y->indptr, Y->indices, Y->rows, Y->cols,
                       Y->nnz, flag_dev);
    ALS_HIP(ctx, hipGetLastError());
    return ALS_OK;
}

}  // namespace als
