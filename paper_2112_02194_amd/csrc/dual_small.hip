// Row classes k <= 4 and 5 <= k <= 8, compiled once each with -DSMALL_G=4 and -DSMALL_G=8 (step: dual_small_step.h).
#include "dual_small_step.h"
#include "dual_walk.h"
#include "row_copy.h"
#include "step_queue.h"
#include "x_rows.h"

#ifndef SMALL_G
#error "compile with -DSMALL_G=8 or -DSMALL_G=4"
#endif

namespace als {

// The two launch forms of a step kernel (see StepGrid): one step per workgroup, or a grid-stride walk from
// step first_blk to the end of the list.
template <int D, int G, bool LOOP>
__global__ __launch_bounds__(64) void dual_small_kernel(const int64_t *__restrict__ indptr,
                                                        const int32_t *__restrict__ indices,
                                                        const float *__restrict__ values,
                                                        const void *__restrict__ Z, float *__restrict__ R,
                                                        int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                        const int32_t *__restrict__ count_ptr, int first_blk,
                                                        int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    constexpr int NR = SmallCfg<D, G>::NR;
    const int count = *count_ptr;
    const int steps = list_steps(count, NR);  // compared with instead of blk * NR, which does not fit beyond the end of a list of 2^31 rows
    int blk = first_blk + blockIdx.x;
    if constexpr (!LOOP) {
        blk = xcd_step(blk, gridDim.x, steps);
        if (blk < steps) dual_small_step<D, G, false>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
    } else {
        for (; blk < steps; blk += gridDim.x) {
            dual_small_step<D, G, false>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R), opaque(ldr), opaque(r0),
                              opaque(list), opaque(count), opaque(err_flag), blk, opaque(lds));
            wave_sync();  // the next step reuses the LDS buffers
        }
    }
}

// The same step with X = R L^-1 taken along (fp32 tables with d >= 64, bf16 tables with d >= 32): the wavefront's rows of R go from registers through LDS
// into x_rows and never to memory, where a pass of its own writes and reads each of them once more.  Epoch of 50M x 50M rows (d =
// 128), 81M of whose 100M solved rows come through here: 132.0 -> 115.2 ms (these kernels 46.0 -> 47.5 ms, the pass over the rows left
// 24.8 -> 4.3 ms); 10M pages: 55.2 -> 54.1 ms; 1M x 1M (d = 64) the two together 402 -> 324 us.
// The matrix stands in LDS once per workgroup (60 KB at d = 128), so the launch is persistent and its wavefronts take their
// steps in turn or, where they get many, from a queue (50M x 50M: 49.7 ms in turn, 47.5 from the queue; 378 000 rows of 5 to 8 entries, d = 64:
// 142 us in turn, 237 from a queue, whose counters all wavefronts ask at the end).  List entry, row descriptor and column id of the next step are loaded while a step is solved: lane
// l = 16 p + a of the wavefront keeps those of entry slot a of tile p.
// bf16 tables: 20M x 20M rows of 6 entries (d = 128) 10.8 -> 9.9 ms and 6.7 -> 0.02 ms of the pass, the epoch 31.6 -> 24.3; 3M x 2M (d = 64)
// 2.53 -> 2.18 ms, 2M x 3M (d = 32) 1.59 -> 1.35 ms (with 8 < k <= 32, dual_walk.h).
// What bounds it: HBM (50M rows of 1 to 8 entries, fp32: 5.0 TB/s with the rows of Z, ids and X; two wavefronts per SIMD, three with bf16).
template <int D, int G, bool ZB> struct SmallXCfg {
    static constexpr int THREADS = ZB ? 768 : 512;
    using M = XMatrix<D, ZB>;
    typedef typename std::conditional<ZB, uint16_t, float>::type elem;
    static constexpr int RLD = row_copy_stride(D);  // of the copy of R
    static constexpr int WAVE_FLOATS = SmallCfg<D, G>::OFF_META;
    static_assert(16 * RLD <= SmallCfg<D, G>::MAIN, "sixteen rows of R take the place of a tile's entries");
    static constexpr size_t LDS_BYTES = M::BYTES + (THREADS / 64) * WAVE_FLOATS * sizeof(float);
};

template <int D, int G, bool ZB>
__global__ __launch_bounds__((SmallXCfg<D, G, ZB>::THREADS)) void dual_small_x_kernel(
    const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices, const float *__restrict__ values, const void *__restrict__ Z,
    typename SmallXCfg<D, G, ZB>::elem *__restrict__ X, int64_t ldx, int64_t r0, const int32_t *__restrict__ list,
    const int32_t *__restrict__ count_ptr, const float *__restrict__ LinvT, int32_t *__restrict__ queue, int32_t *__restrict__ err_flag) {
    using C = SmallCfg<D, G>;
    using CX = SmallXCfg<D, G, ZB>;
    using M = typename CX::M;
    constexpr int NR = C::NR, NJ = z_pieces<D, ZB>(), CPL = columns_per_lane(D), NK = D / 32;
    extern __shared__ float shared[];
    const int count = *count_ptr;
    if (count <= 0) return;
    char *mat = (char *)shared;
    M::template fill<CX::THREADS>(mat, LinvT, threadIdx.x);
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float *lds = (float *)(mat + M::BYTES) + wave * CX::WAVE_FLOATS;
    const int slot = lane % G;
    X += r0 * ldx;
    indptr += r0;

    StepQueue steps = step_queue(queue, list_steps(count, NR), blockIdx.x, gridDim.x, wave, CX::THREADS / 64);
    auto next_step = [&]() {
        return steps.next([](const int32_t *counter) { return __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)); },
                          [&](int32_t *counter, int n) {
                              int at = 0;
                              if (lane == 0) at = atomicAdd(counter, n);
                              return __builtin_amdgcn_readfirstlane(at);
                          });
    };
    auto place = [&](int blk) {  // place in the list of the row of which this lane keeps an entry
        return (unsigned)blk * NR + (unsigned)(lane / G);
    };
    auto row_of = [&](int blk) { return list[place(blk) < (unsigned)count ? place(blk) : (unsigned)count - 1u]; };

    int blk = next_step();
    if (blk < 0) return;
    int next = next_step();
    int32_t rel = row_of(blk), rel_next = next < 0 ? rel : row_of(next);
    int64_t b = indptr[rel];
    int k = place(blk) < (unsigned)count ? (int)(indptr[rel + 1] - b) : 0;
    int64_t at = b + (slot < k ? slot : 0);  // a row of the list has k >= 1: always in range
    int32_t id = indices[at];
    float y = slot < k ? (values ? values[at] : 1.f) : 0.f;
    for (;;) {
        // ---- gather, all loads of the step
        float4 z[4][NJ];
        {
            const int a = lane & 15, q = lane >> 4;
            const int own = slot < k ? id : -1;
            int32_t ids[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) ids[p] = __shfl(own, 16 * p + a);
#pragma unroll
            for (int p = 0; p < 4; ++p) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[p][j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (ids[p] >= 0) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) z[p][j] = load_piece<D, ZB>(Z, ids[p], j, q);
                }
            }
        }
        // ---- the next step's row descriptors, the list entries of the one after it
        const int64_t b_next = indptr[rel_next], e_next = indptr[rel_next + 1];
        const int after = next < 0 ? -1 : next_step();
        const int32_t rel_after = after < 0 ? rel_next : row_of(after);

        small_solve<D, G, ZB>(z, y, lds, err_flag);

        // ---- the next step's column ids
        const int k_next = next >= 0 && place(next) < (unsigned)count ? (int)(e_next - b_next) : 0;
        const int64_t at_next = b_next + (slot < k_next ? slot : 0);
        const int32_t id_next = indices[at_next];
        const float y_next = slot < k_next ? (values ? values[at_next] : 1.f) : 0.f;

        float r[NR][CPL];
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
            for (int c = 0; c < CPL; ++c) r[n][c] = 0.f;
        small_rows<D, G, ZB>(z, lds, [&](int n) { return __builtin_amdgcn_readlane(k, n * G); }, [&](int n, const float (&v)[CPL]) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) r[n][c] = v[c];
        });
        wave_sync();
        // ---- X = R L^-1 of the wavefront's rows (with G = 8 the rows 8 .. 15 of the tile are whatever lies there)
        if (holds_columns(D, lane)) {
#pragma unroll
            for (int n = 0; n < NR; ++n) {
                float *to = lds + row_copy_place(D, n, lane);
                if constexpr (CPL == 2) *(float2 *)to = make_float2(r[n][0], r[n][1]);
                else *to = r[n][0];
            }
        }
        wave_sync();
        const int a = lane & 15, q = lane >> 4;
        bf16x8 xp[1][M::PARTS][NK];
#pragma unroll
        for (int kb = 0; kb < NK; ++kb) {
            const float *src = lds + a * CX::RLD + 32 * kb + 8 * q;
            bf16x8 part[M::PARTS];
            M::cut(*(const float4 *)src, *(const float4 *)(src + 4), part);
#pragma unroll
            for (int t = 0; t < M::PARTS; ++t) xp[0][t][kb] = part[t];
        }
        const int32_t my_rel = __shfl(rel, a * G & 63);
        const int my_k = __shfl(k, a * G & 63);  // by all lanes: a lane that is masked out gives nothing
        const bool mine = a < NR && my_k > 0;
        typename CX::elem *dst = X + my_rel * ldx + 8 * q;
        x_rows<D, ZB, 1>(mat, xp, [&](int, int P, const floatx4 (&v)[2]) {
            if (mine) store_x8<ZB>(dst + 32 * P, v);
        });
        if (next < 0) break;
        wave_sync();  // the next step reuses the LDS buffers
        blk = next;
        next = after;
        rel = rel_next;
        rel_next = rel_after;
        k = k_next;
        id = id_next;
        y = y_next;
    }
}

template <int D, bool ZB>
static als_status launch_small_x_typed(als_ctx *ctx, const als_csr *Y, const void *Z, void *X, int64_t ldx, int64_t r0, const int32_t *list,
                                       const int32_t *count_dev, WalkSize w, const float *LinvT, int32_t *queue, int32_t *err,
                                       hipStream_t s) {
    using CX = SmallXCfg<D, SMALL_G, ZB>;
    static const hipError_t attr = hipFuncSetAttribute((const void *)dual_small_x_kernel<D, SMALL_G, ZB>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)CX::LDS_BYTES);  // once per process
    ALS_HIP(ctx, attr);
    constexpr int64_t WAVES = CX::THREADS / 64, PER_CU = 160 * 1024 / CX::LDS_BYTES;
    const int64_t most = w.num_cu * PER_CU, wanted = ((w.hint < 0 ? w.capacity : std::min(w.hint, w.capacity)) + WAVES - 1) / WAVES;
    const unsigned blocks = (unsigned)(std::max<int64_t>(1, std::min(most, wanted)) + 7) / 8 * 8;
    hipLaunchKernelGGL((dual_small_x_kernel<D, SMALL_G, ZB>), dim3(blocks), dim3(CX::THREADS), CX::LDS_BYTES, s, Y->indptr, Y->indices,
                       Y->values, Z, (typename CX::elem *)X, ldx, r0, list, count_dev, LinvT, queue, err);
    return ALS_OK;
}

#if SMALL_G == 8
als_status launch_dual_small8_x(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, void *X, int64_t ldx, int64_t r0,
                                const int32_t *list, const int32_t *count_dev, WalkSize w, const float *LinvT, int32_t *queue, int32_t *err, hipStream_t s) {
#else
als_status launch_dual_small4_x(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, void *X, int64_t ldx, int64_t r0,
                                const int32_t *list, const int32_t *count_dev, WalkSize w, const float *LinvT, int32_t *queue, int32_t *err, hipStream_t s) {
#endif
#define ALS_SMALL_CASE(dd, zb) launch_small_x_typed<dd, zb>(ctx, Y, Z, X, ldx, r0, list, count_dev, w, LinvT, queue, err, s)
    if (zb16) return d == 128 ? ALS_SMALL_CASE(128, true) : (d == 64 ? ALS_SMALL_CASE(64, true) : ALS_SMALL_CASE(32, true));
    return d == 128 ? ALS_SMALL_CASE(128, false) : ALS_SMALL_CASE(64, false);
#undef ALS_SMALL_CASE
}

template <int D>
static void launch_small_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                               const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
    using C = SmallCfg<D, SMALL_G>;
    if (g.known > 0)
        hipLaunchKernelGGL((dual_small_kernel<D, SMALL_G, false>), dim3(g.known), dim3(64),
                           C::LDS_FLOATS * sizeof(float), s, Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list,
                           count_dev, 0, err);
    if (g.rest > 0)
        hipLaunchKernelGGL((dual_small_kernel<D, SMALL_G, true>), dim3(g.rest), dim3(64),
                           C::LDS_FLOATS * sizeof(float), s, Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list,
                           count_dev, (int)g.known, err);
}

#if SMALL_G == 8
void launch_dual_small8(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#else
void launch_dual_small4(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#endif
    if (d == 16) launch_small_typed<16>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);
    else launch_small_typed<32>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);
}

}  // namespace als
