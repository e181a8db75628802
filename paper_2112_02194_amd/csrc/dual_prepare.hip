// Dual (k x k) form of the row update of the paper's Eq. 4 for rows with few stored entries.
//
// With B = alpha*G + lambda*I = L L^T (one shared d x d factorisation per half-epoch) and
// z_i = L^{-1} v_i, the normal equations of a row with entries I (|I| = k) become
//     A = B + V_I^T V_I = L (I_d + Z_I^T Z_I) L^T ,
// and the push-through identity (I_d + Z^T Z)^{-1} Z^T = Z^T (I_k + Z Z^T)^{-1} gives
//     x_u = A^{-1} V_I^T y = L^{-T} Z_I^T t ,   (I_k + Z_I Z_I^T) t = y .
// This is the same minimiser of Eq. 3 as the d x d system (exact algebra, no approximation), but
// costs O(k^2 d + k^3) per row instead of O(k d^2 + d^3), and the k x k matrix has eigenvalues in
// [1, 1 + k/alpha], so fp32 is comfortable.  Steps:
//   factor_kernel     B -> L^{-1} in fp64 (one workgroup, up to 8192 rows beside the sort: solve_rows.hip), stored fp32
//   transform_kernel  Z = V L^{-T}   (fp32 MFMA, table-sized workspace)
//   row kernels       by class of k (fixed by measurement on MI355X): all gather Z_I into MFMA operand
//                     registers, straight or by way of LDS, form S = I + Z_I Z_I^T on the matrix cores,
//                     solve the k x k system on the vector ALU, then r = Z_I^T t
//       dual_small_kernel  k <= 4 and 5 <= k <= 8: several rows share one 16-entry MFMA tile (dual_small_x_kernel takes
//                          the last step along, and so do dual_rows_x_kernel and dual_multi_x_kernel for bf16 tables)
//       dual_rows_kernel   8 < k <= 16: four rows per wavefront, one lane per row of S, gather through LDS
//       dual_multi_kernel  16 < k <= 32: four rows per wavefront, S in two blocks of 16
//       dual_triple_kernel 32 < k <= 48 (d >= 64): four rows per wavefront, S in three blocks of 16
//       dual_wide_kernel, dual_wide_rest_kernel  48 < k <= 128 (d = 128; k <= 64 at d = 64): one row per wavefront, S as a
//                          lower triangle in LDS, blocked elimination with MFMA trailing updates
//       dual_few_kernel    all of them, where the lists are short together
//                          (conjugate gradients: dual_wide_kernel for every class)
//   transform_lists_kernel, transform_kernel (d = 16, fp32 with d = 32)
//                     X = R L^{-1}   (rows r -> L^{-T} r), rounding to the table's element type
#include "dual_common.h"
#include "dual_few.h"
#include "dual_walk.h"
#include "dual_wide_rest.h"
#include "factor.h"
#include "step_queue.h"
#include "x_rows.h"

namespace als {

// per-class launchers (`count_dev`: device address of the list's length; `g`, `w`: see StepGrid, WalkSize; `zb16`: Z is bf16), fp32 Z with
// d = 16 or 32
void launch_dual_small4(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s);
void launch_dual_small8(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s);
// the other tables, with X = R L^-1 taken along; `queue`: see StepQueue, zero when the launch begins
als_status launch_dual_small4_x(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, void *X, int64_t ldx, int64_t r0,
                                const int32_t *list, const int32_t *count_dev, WalkSize w, const float *LinvT, int32_t *queue,
                                int32_t *err, hipStream_t s);
als_status launch_dual_small8_x(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, void *X, int64_t ldx, int64_t r0,
                                const int32_t *list, const int32_t *count_dev, WalkSize w, const float *LinvT, int32_t *queue,
                                int32_t *err, hipStream_t s);
// fp32 Z
void launch_dual_k16(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                     const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s);
void launch_dual_multi2(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s);
// bf16 Z, with X = R L^-1 taken along
void launch_dual_k16_x(int d, const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list,
                       const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s);
void launch_dual_multi2_x(int d, const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list,
                          const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s);
// direct solver
void launch_dual_triple(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s);
#define ALS_DECL_WIDE(kt)                                                                                          \
    als_status launch_dual_wide##kt(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R,     \
                                    int64_t ldr, int64_t r0, const int32_t *list, const int32_t *count_dev,        \
                                    StepGrid g, int32_t *err, const WideSolver &ws, hipStream_t s);
ALS_DECL_WIDE(3) ALS_DECL_WIDE(4) ALS_DECL_WIDE(5) ALS_DECL_WIDE(6) ALS_DECL_WIDE(7) ALS_DECL_WIDE(8)
#undef ALS_DECL_WIDE

// ---------------------------------------------------------------------------------------------- factor
template <int D>
__global__ __launch_bounds__(FACTOR_THREADS) void factor_kernel(const float *__restrict__ G, float alpha, float lambda,
                                                                float *__restrict__ Linv, float *__restrict__ LinvT,
                                                                int32_t *__restrict__ err_flag) {
    extern __shared__ double fa[];
    factor<D>(G, alpha, lambda, Linv, LinvT, err_flag, fa);
}

// ---------------------------------------------------------------------------------------------- transform
// Out[r][:] = In[r][:] * M for rows r in [r0, r1) (only rows with 0 < k <= k_max stored entries when
// indptr is given), M fp32 [D x D] row-major and triangular: UPPER = true means M[j][c] = 0 for j > c
// (M = L^{-T}), UPPER = false means M[j][c] = 0 for j < c (M = L^{-1}).  In may be bf16 or fp32, Out
// fp32 or bf16; Out may be the same buffer as In (a wavefront reads its rows completely before it
// writes them, and no other wavefront touches them).
//
// A wavefront owns TM table rows at a time and all D output columns.  Lane (m, kq) streams along row
// m: for the contraction block kb (TM input columns) it holds the BW = TM/KS consecutive columns
// TM*kb + BW*kq .. of its row, loaded straight from global memory as 16-byte pieces; step i of the
// block contracts column TM*kb + BW*kq + i (A and B operands only have to agree on that mapping).
// The transposed matrix Mt (Mt[c][j] = M[j][c]; the factorisation leaves both) sits in LDS (one copy per
// workgroup, padded rows) and supplies the B operands; blocks that only meet zeros of the triangular matrix
// are skipped.
//
// GATHER (Z = V L^{-T} for few entries of a large table): "row" p of the pass is entry p of the CSR arrays, its input
// the table row ids[p], its output row p of Z; the range of p is read from *first and *last on the device, and
// entry_ids[p] = p becomes the index by which the row kernels find their entries.
struct Gather {
    const int32_t *ids;
    const int64_t *first, *last;
    int32_t *entry_ids;
    int64_t limit;  // rows of Z: an indptr that claims more entries is cut off
    __device__ int64_t begin() const { return *first < 0 ? 0 : *first; }
    __device__ int64_t end() const { return *last < limit ? *last : limit; }
};
template <int D> struct XfCfg {
    using GE = Geo<D>;
    static constexpr int TM = GE::TM, KS = GE::KS, NB = D / TM, BW = TM / KS, MLD = D + 4;
    static constexpr size_t LDS_BYTES = (size_t)D * MLD * sizeof(float);
};

template <int D, bool IN_BF16, bool OUT_BF16, bool UPPER, bool GATHER>
__global__ __launch_bounds__(256) void transform_kernel(const void *In, int64_t ldi, void *Out, int64_t ldo,
                                                        const float *__restrict__ Mt, int64_t r0, int64_t r1,
                                                        const int64_t *__restrict__ indptr, int64_t k_max, Gather ga) {
    using C = XfCfg<D>;
    constexpr int TM = C::TM, NB = C::NB, BW = C::BW, MLD = C::MLD, ACC = Geo<D>::ACC;
    typedef typename AccT<ACC>::type acc_t;
    extern __shared__ float MT[];  // MT[c * MLD + j] = M[j][c]
#pragma unroll 4
    for (int e = threadIdx.x; e < D * D / 4; e += 256) *(float4 *)(MT + e / (D / 4) * MLD + 4 * (e % (D / 4))) = ((const float4 *)Mt)[e];
    if constexpr (GATHER) {
        r0 = ga.begin();
        r1 = ga.end();
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane % TM, kq = lane / TM;
    const int64_t ntiles = (r1 - r0 + TM - 1) / TM;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < ntiles; tile += nwaves) {
        const int64_t base = r0 + tile * TM, row = base + m;
        int64_t src = row;
        if constexpr (GATHER) {
            src = row < r1 ? ga.ids[row] : 0;
            if (kq == 0 && row < r1) ga.entry_ids[row] = (int32_t)row;
        }
        float a[NB][BW];
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
            for (int i4 = 0; i4 < BW / 4; ++i4) {
                float x[4] = {0.f, 0.f, 0.f, 0.f};
                if (row < r1) load_vec<4, IN_BF16>(In, src * ldi + TM * kb + BW * kq + 4 * i4, x);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[kb][4 * i4 + c] = x[c];
            }
        // which of this lane's ACC output rows are written (only rows solved in the dual form)
        bool keep[ACC];
#pragma unroll
        for (int v = 0; v < ACC; ++v) {
            const int64_t r = base + acc_row<D>(v, lane);
            keep[v] = r < r1;
            if (keep[v] && indptr) {
                const int64_t k = indptr[r + 1] - indptr[r];
                keep[v] = k > 0 && k <= k_max;
            }
        }
#pragma unroll
        for (int J = 0; J < NB; ++J) {
            acc_t acc;
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[v] = 0.f;
#pragma unroll
            for (int kb = 0; kb < NB; ++kb) {
                if (UPPER ? (kb <= J) : (kb >= J)) {  // compile-time after unrolling
                    const float *bp = MT + (TM * J + m) * MLD + TM * kb + BW * kq;
#pragma unroll
                    for (int i4 = 0; i4 < BW / 4; ++i4) {
                        const float4 b = *(const float4 *)(bp + 4 * i4);
                        acc = mfma<D>(a[kb][4 * i4 + 0], b.x, acc);
                        acc = mfma<D>(a[kb][4 * i4 + 1], b.y, acc);
                        acc = mfma<D>(a[kb][4 * i4 + 2], b.z, acc);
                        acc = mfma<D>(a[kb][4 * i4 + 3], b.w, acc);
                    }
                }
            }
            // acc[v] = Out[base + acc_row(v)][TM*J + m]
#pragma unroll
            for (int v = 0; v < ACC; ++v)
                if (keep[v]) store_elem<OUT_BF16>(Out, (base + acc_row<D>(v, lane)) * ldo + TM * J + m, acc[v]);
            __builtin_amdgcn_sched_barrier(0);  // keep the next column tile's operand reads from piling up
        }
    }
}

// ---------------------------------------------------------------------------------------------- transform, bf16 output
// Z = V L^-T for bf16 tables (d >= 32), where Z is bf16 too: on the bf16 matrix cores,
// which turns the pass from matrix-core-bound (fp32 instruction) into HBM-bound.  M is cut once per workgroup
// into hi = bf16(M) and lo = bf16(M - hi) (LDS, transposed); the table's rows are exact operands (two products
// per step: x hi + x lo).  The error of the cut, 2^-17 relative, is far below the bf16 rounding of the output.
// The roles of the operands are swapped against transform_kernel: the matrix supplies the M dimension
// (output columns) and the table rows the N dimension, so that a lane ends up with 16 consecutive output
// columns of ONE table row (the output columns are assigned to the instruction's row index in the order
// that makes them consecutive) and stores them as two 16-byte pieces.
template <int D> struct Xf16Cfg {
    static constexpr int MLD = D + 8;  // bf16 elements per LDS row (rows stay 16-byte aligned)
    static constexpr size_t LDS_BYTES = (size_t)2 * D * MLD * sizeof(uint16_t);
};

template <int D, bool GATHER>
__global__ __launch_bounds__(256, 2) void transform16_kernel(const uint16_t *__restrict__ In, int64_t ldi,
                                                          uint16_t *__restrict__ Out, int64_t ldo,
                                                          const float *__restrict__ Mt, int64_t r0, int64_t r1, Gather ga) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int MLD = Xf16Cfg<D>::MLD, NKB = D / 16, NJB = D / 32;
    extern __shared__ uint16_t mt[];  // hi: mt[c * MLD + j] = bf16(M[j][c]); lo: the same at offset D * MLD
#pragma unroll 4
    for (int e = threadIdx.x; e < D * D / 4; e += 256) {
        const float4 v = ((const float4 *)Mt)[e];
        const uint32_t h0 = pack_nearest(v.x, v.y), h1 = pack_nearest(v.z, v.w);
        uint16_t *at = mt + e / (D / 4) * MLD + 4 * (e % (D / 4));
        *(uint2 *)at = make_uint2(h0, h1);
        *(uint2 *)(at + D * MLD) = make_uint2(pack_nearest(v.x - __uint_as_float(h0 << 16), v.y - __uint_as_float(h0 & 0xffff0000u)),
                                              pack_nearest(v.z - __uint_as_float(h1 << 16), v.w - __uint_as_float(h1 & 0xffff0000u)));
    }
    if constexpr (GATHER) {
        r0 = ga.begin();
        r1 = ga.end();
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, kq = lane >> 5;
    // output column (inside a block of 32) that this lane supplies as row n of the matrix operand
    const int pi = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
    const int64_t ntiles = (r1 - r0 + 31) / 32;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < ntiles; tile += nwaves) {
        const int64_t row = r0 + tile * 32 + n;
        const bool keep = row < r1;
        // this lane's share of its row: columns 16 kb + 8 kq .., operands as they are
        int64_t src = row;
        if constexpr (GATHER) {
            src = row < r1 ? ga.ids[row] : 0;
            if (kq == 0 && row < r1) ga.entry_ids[row] = (int32_t)row;
        }
        bf16x8 xh[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if (keep) w = *(const u32x4 *)(In + src * ldi + 16 * kb + 8 * kq);
            xh[kb] = __builtin_bit_cast(bf16x8, w);
        }
#pragma unroll
        for (int J = 0; J < NJB; ++J) {
            floatx16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
            const uint16_t *mrow = mt + (32 * J + pi) * MLD + 8 * kq;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                if (kb <= 2 * J + 1) {  // compile-time after unrolling: other steps only meet zeros
                    const bf16x8 mh = *(const bf16x8 *)(mrow + 16 * kb), ml = *(const bf16x8 *)(mrow + D * MLD + 16 * kb);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mh, xh[kb], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ml, xh[kb], acc, 0, 0, 0);
                }
            }
            // acc[v] = Out[row][32 J + 16 kq + v]
            if (keep) {
                u32x4 lo4, hi4;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    lo4[w] = pack_nearest(acc[2 * w], acc[2 * w + 1]);
                    hi4[w] = pack_nearest(acc[8 + 2 * w], acc[8 + 2 * w + 1]);
                }
                u32x4 *dst = (u32x4 *)(Out + row * ldo + 32 * J + 16 * kq);
                dst[0] = lo4;
                dst[1] = hi4;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- X = R L^-1 of class lists
// x_rows.h over the rows of some class lists, 32 rows per wavefront at a time, fp32 tables (d >= 64) in place, bf16 tables (d >= 32)
// from the fp32 rows of R.  fp32: 0.375 of the fp32 instruction's matrix-core time, which leaves the pass to the table read and
// write (for Z = V L^-T the fp32 kernel above measured faster, 24.4 against 25.9 ms per epoch of 50M x 50M).
// What bounds it: HBM (4.5 TB/s of rows read and written); in short calls the chain of counts, list entries, rows and the matrix that every
// workgroup lays out for itself.  Rows of 12 entries, workgroups for all that the lists' capacities come to, eight wavefronts each / as
// it is (tile_grid), us: d = 128, bf16 9000 rows 10.3 / 7.6, 15 000 11.2 / 7.9, 30 000 12.2 / 9.2, fp32 9000 13.4 / 9.6, 30 000 15.2 / 12.1, 60 000
// 19.0 / 17.2; d = 64, fp32, 9000 7.9 / 6.0.
struct XLists {
    const int32_t *list[10], *count[10];  // beyond n: the first once more
    int n;
};

template <int D, bool BF, int T>
__global__ __launch_bounds__(T, 2) void transform_lists_kernel(const float *R, int64_t ldr,
                                                                         typename std::conditional<BF, uint16_t, float>::type *X, int64_t ldx,
                                                                         const float *__restrict__ LinvT, int64_t r0, XLists xl) {
    using M = XMatrix<D, BF>;
    constexpr int NK = D / 32;
    extern __shared__ char mat[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), a = lane & 15, q = lane >> 4;
    R += r0 * ldr;
    X += r0 * ldx;
    const int nwaves = (int)gridDim.x * (T / 64);
    int counts[10], total = 0;  // all loads at once
#pragma unroll
    for (int c = 0; c < 10; ++c) counts[c] = *xl.count[c];
#pragma unroll
    for (int c = 0; c < 10; ++c) {
        if (c >= xl.n) counts[c] = 0;
        total += list_steps(counts[c], 32);
    }
    int tile = (int)blockIdx.x * (T / 64) + wave;  // counted from the first tile of the first list
    int32_t rel[2] = {0, 0};
    bool have[2] = {false, false};
    float4 raw[2][NK][2];
    auto load = [&] {
        const int32_t *list = nullptr;
        int count = 0, in_list = 0, first = 0;
#pragma unroll
        for (int c = 0; c < 10; ++c) {
            const bool here = tile >= first;  // the last list that begins at or before the tile, and is not empty
            const int steps = list_steps(counts[c], 32);
            list = here && steps > 0 ? xl.list[c] : list;
            count = here && steps > 0 ? counts[c] : count;
            in_list = here && steps > 0 ? tile - first : in_list;
            first += steps;
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const unsigned item = 32u * (unsigned)in_list + 16u * n + (unsigned)a;
            have[n] = item < (unsigned)count;
            rel[n] = list[have[n] ? item : (unsigned)count - 1u];
        }
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
                const float *src = R + rel[n] * ldr + 32 * kb + 8 * q;
                raw[n][kb][0] = *(const float4 *)src;
                raw[n][kb][1] = *(const float4 *)(src + 4);
            }
    };
    if (tile < total) load();  // the first rows are on their way while the matrix is laid out
    M::template fill<T>(mat, LinvT, threadIdx.x);
    __syncthreads();
    while (tile < total) {
        bf16x8 xp[2][M::PARTS][NK];
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
                bf16x8 part[M::PARTS];
                M::cut(raw[n][kb][0], raw[n][kb][1], part);
#pragma unroll
                for (int t = 0; t < M::PARTS; ++t) xp[n][t][kb] = part[t];
            }
        x_rows<D, BF, 2>(mat, xp, [&](int n, int P, const floatx4 (&v)[2]) {
            if (have[n]) store_x8<BF>(X + rel[n] * ldx + 32 * P + 8 * q, v);
        });
        tile += nwaves;
        if (tile < total) load();
    }
}

// XMatrix for the kernels that read it from device memory
template <int D> __global__ __launch_bounds__(64) void x_matrix_kernel(const float *__restrict__ LinvT, char *__restrict__ mat) {
    XMatrix<D, true>::template fill<XMatrix<D, true>::BLOCKS * 64>(mat, LinvT, blockIdx.x * 64 + threadIdx.x);
}

// ---------------------------------------------------------------------------------------------- launchers
// Rows of 48 < k <= 128 that one launch takes for several classes where an earlier call saw so few (or that no hint announced).  That launch has
// the registers and the LDS of its largest class, one wavefront per SIMD with fp32 at d = 128, so a row takes longer in it, but a
// class by itself ends with the chain of its last rows.  Calls that fold rows in, 4 / 8 / 16 / 32 rows per compute unit, us: 300 000 rows,
// 3M items, d = 128, bf16 829 / 808 / 809 / 817; 150 000 rows, 1M items, d = 128, fp32 763 / 762 / 749 / 749, 300 000 1010 / 988 / 987 / 989, 1M
// 2213 / 2212 / 2202 / 2200; 600 000 bf16 812 / 812 / 795 / 797.
inline int64_t wide_rest_limit(int num_cu) { return 16 * (int64_t)num_cu; }

int dual_supported_max_k(int d) { return d < 128 ? (d < 64 ? d : 64) : 128; }

// bf16 tables with d >= 32: Z is stored as bf16 too (one more rounding, to the tables' own element type, of a
// table that is only ever used to solve rows whose result is rounded to bf16 anyway; half the gather
// traffic, and a row piece is a matrix-core operand as loaded).  At d = 16 a row is shorter than one
// 32-column matrix-core step and Z stays fp32.
template <int D, bool BF16> constexpr bool z_is_bf16() { return BF16 && D >= 32; }

// Part 1 (needs no row classification): factorise B and build Z = V L^{-T}, of the whole table, or (`entries`) of
// the table rows that the entries of rows [r0, r1) name, in the order of the entries.
template <int D, bool BF16>
static als_status dual_prepare_typed(als_ctx *ctx, const als_table *V, const float *G, const als_params *prm,
                                     const als_csr *entries, int64_t r0, int64_t r1, bool factored, hipStream_t s) {
    constexpr bool ZB = z_is_bf16<D, BF16>();
    const int64_t zrows = entries ? entries->nnz : V->rows;
    als_status st = ensure(ctx, ctx->ztable, (size_t)zrows * D * (ZB ? 2 : 4));
    if (st != ALS_OK) return st;
    Gather ga = {nullptr, nullptr, nullptr, nullptr, 0};
    if (entries) ga = {entries->indices, entries->indptr + r0, entries->indptr + r1, (int32_t *)ctx->entry_ids.p, entries->nnz};
    float *Linv = (float *)((char *)ctx->small.p + SM_FACTOR), *LinvT = Linv + 128 * 128;
    int32_t *err = (int32_t *)((char *)ctx->small.p + SM_COUNTERS) + 2;
    timer_begin(ctx, T_TRANSFORM, s);
    if (!factored) {
        constexpr size_t factor_lds = FactorCfg<D>::LDS_BYTES;
        static const hipError_t attr_f = hipFuncSetAttribute((const void *)factor_kernel<D>,
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)factor_lds);
        ALS_HIP(ctx, attr_f);
        hipLaunchKernelGGL(factor_kernel<D>, dim3(1), dim3(FACTOR_THREADS), factor_lds, s, G, prm->alpha, prm->lambda, Linv, LinvT,
                           err);
    }
    const unsigned tblocks = (unsigned)std::min<int64_t>(1024, std::max<int64_t>(1, (zrows + 127) / 128));
    auto transform = [&](auto gather) {  // L^{-1} is the transpose of the matrix applied
        constexpr bool GA = decltype(gather)::value;
        if constexpr (ZB) {
            static const hipError_t attr = hipFuncSetAttribute((const void *)transform16_kernel<D, GA>,
                                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                                               (int)Xf16Cfg<D>::LDS_BYTES);  // once per process
            if (attr == hipSuccess)
                hipLaunchKernelGGL((transform16_kernel<D, GA>), dim3(tblocks), dim3(256), Xf16Cfg<D>::LDS_BYTES, s,
                                   (const uint16_t *)V->data, V->ld, (uint16_t *)ctx->ztable.p, (int64_t)D, (const float *)Linv,
                                   (int64_t)0, V->rows, ga);
            return attr;
        } else {
            static const hipError_t attr = hipFuncSetAttribute((const void *)transform_kernel<D, BF16, false, true, GA>,
                                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                                               (int)XfCfg<D>::LDS_BYTES);  // once per process
            if (attr == hipSuccess)
                hipLaunchKernelGGL((transform_kernel<D, BF16, false, true, GA>), dim3(tblocks), dim3(256), XfCfg<D>::LDS_BYTES, s,
                                   V->data, V->ld, ctx->ztable.p, (int64_t)D, (const float *)Linv, (int64_t)0, V->rows,
                                   (const int64_t *)nullptr, (int64_t)0, ga);
            return attr;
        }
    };
    ALS_HIP(ctx, entries ? transform(std::true_type{}) : transform(std::false_type{}));
    timer_end(ctx, s);
    ALS_HIP(ctx, hipGetLastError());
    return ALS_OK;
}

// Part 2: the row kernels of the k-classes, then X = R L^{-1} on the rows they solved.  Every class is
// launched (its kernel finds the length of its list in device memory); `caps` bounds the lists, `hints` holds
// the lengths seen by the previous call on the same matrix, or -1.
template <int D, bool BF16>
static als_status dual_rows_typed(als_ctx *ctx, const als_csr *Y, als_table *X, int64_t r0, int64_t r1,
                                  int dual_max, const als_params *prm, const int32_t *const lists[10],
                                  const int32_t *const counts_dev[10], const int64_t caps[10], const int hints[10],
                                  hipStream_t s) {
    float *R = (float *)X->data;
    int64_t ldr = X->ld;
    if (BF16) {
        als_status st = ensure(ctx, ctx->rtable, (size_t)(r1 - r0) * D * sizeof(float));
        if (st != ALS_OK) return st;
        R = (float *)ctx->rtable.p - r0 * D;  // row u lives at rtable[(u - r0) * D]
        ldr = D;
    }
    const float *LinvT = (const float *)((char *)ctx->small.p + SM_FACTOR) + 128 * 128;  // transpose of the matrix applied
    int32_t *err = (int32_t *)((char *)ctx->small.p + SM_COUNTERS) + 2;
    int32_t *queue = (int32_t *)((char *)ctx->small.p + SM_QUEUE);
    const void *Z = ctx->ztable.p;
    constexpr bool zb16 = z_is_bf16<D, BF16>(), X_LISTS = zb16 || (!BF16 && D >= 64);
    bool is_x[10] = {false};  // classes whose rows leave their kernel as X
    als_status stb = ALS_OK;
    // workgroups of class `cls` whose kernel takes `rpw` rows per step
    auto grid = [&](int cls, int rpw) {
        const int64_t cap = (caps[cls] + rpw - 1) / rpw;
        const int64_t hint = hints[cls] < 0 ? -1 : ((int64_t)hints[cls] + rpw - 1) / rpw;
        return step_grid(ctx->num_cu, 64, cap, hint, 32, rpw > 1 ? 1 << 24 : 1 << 22);  // one wavefront per workgroup
    };
    auto walk = [&](int cls, int rpw) {
        return WalkSize{ctx->num_cu, (caps[cls] + rpw - 1) / rpw, hints[cls] < 0 ? -1 : ((int64_t)hints[cls] + rpw - 1) / rpw};
    };
#define ALS_TIMED_CLASS(slot, cls, rpw, call)           \
    if (caps[cls] > 0 && stb == ALS_OK) {               \
        const StepGrid g = grid(cls, rpw);              \
        timer_begin(ctx, slot, s);                      \
        call;                                           \
        timer_end(ctx, s);                              \
    }
    // conjugate gradients on the k x k systems (Section 4.5's solver): every class goes through the
    // one-row-per-wavefront kernel, the classes up to k = 32 through its smallest instance
    const WideSolver ws = {prm->solver == ALS_SOLVER_CG, prm->cg_max_iters > 0 ? prm->cg_max_iters : 2 * D,
                           prm->cg_tol > 0.f ? prm->cg_tol : 1e-6f};
    FewLists few;
    int64_t steps = 0, listed = 0;  // all, and those in the common launch
    const bool own_triple = D >= 64 && !ws.cg && hints[2] >= few_triple_rows(D, zb16);
    for (int c = 0; c < 10; ++c) {
        few.list[c] = lists[c];
        few.count[c] = counts_dev[c];
        few.start[c] = (int32_t)std::min<int64_t>(listed, INT32_MAX);
        const int64_t n = (caps[c] + FEW_ROWS[c] - 1) / FEW_ROWS[c];
        steps += n;
        listed += c == 2 && own_triple ? 0 : n;
    }
    few.start[10] = (int32_t)std::min<int64_t>(listed, INT32_MAX);
    if (!ws.cg && steps <= FEW_STEPS) {
        if constexpr (D >= 64) {
            if (own_triple) {
                ALS_TIMED_CLASS(T_DUAL_CLASS0 + 2, 2, 4, (launch_dual_triple(D, Y, Z, zb16, R, ldr, r0, lists[2], counts_dev[2], walk(2, 4), err, s)))
            }
        }
        if (listed > 0) {
            timer_begin(ctx, T_DUAL_CLASS0, s);
            stb = launch_dual_few(ctx, D, Y, Z, zb16, R, ldr, r0, few, err, s);
            timer_end(ctx, s);
        }
    } else {
    if (ws.cg) {
        if constexpr (D < 64) return fail(ctx, ALS_EINVAL, "conjugate gradients on the dual systems need d >= 64");
        ALS_TIMED_CLASS(T_DUAL_CLASS0 + 1, 1, 1, (stb = launch_dual_wide3(ctx, D, Y, Z, zb16, R, ldr, r0, lists[1], counts_dev[1], g, err, ws, s)))
        ALS_TIMED_CLASS(T_DUAL_CLASS0, 0, 1, (stb = launch_dual_wide3(ctx, D, Y, Z, zb16, R, ldr, r0, lists[0], counts_dev[0], g, err, ws, s)))
        ALS_TIMED_CLASS(T_SMALL8, 9, 1, (stb = launch_dual_wide3(ctx, D, Y, Z, zb16, R, ldr, r0, lists[9], counts_dev[9], g, err, ws, s)))
        ALS_TIMED_CLASS(T_SMALL4, 8, 1, (stb = launch_dual_wide3(ctx, D, Y, Z, zb16, R, ldr, r0, lists[8], counts_dev[8], g, err, ws, s)))
    } else {
    if constexpr (zb16) {
    char *xmat = (char *)ctx->small.p + SM_XMATRIX;
    is_x[0] = is_x[1] = true;
    hipLaunchKernelGGL(x_matrix_kernel<D>, dim3(XMatrix<D, true>::BLOCKS), dim3(64), 0, s, LinvT, xmat);
    const XTable x = {(uint16_t *)X->data, X->ld, xmat};
    ALS_TIMED_CLASS(T_DUAL_CLASS0 + 1, 1, 4, (launch_dual_multi2_x(D, Y, Z, x, r0, lists[1], counts_dev[1], walk(1, 4), err, s)))
    ALS_TIMED_CLASS(T_DUAL_CLASS0, 0, 4, (launch_dual_k16_x(D, Y, Z, x, r0, lists[0], counts_dev[0], walk(0, 4), err, s)))
    } else {
    ALS_TIMED_CLASS(T_DUAL_CLASS0 + 1, 1, 4, (launch_dual_multi2(D, Y, Z, R, ldr, r0, lists[1], counts_dev[1], walk(1, 4), err, s)))
    ALS_TIMED_CLASS(T_DUAL_CLASS0, 0, 4, (launch_dual_k16(D, Y, Z, R, ldr, r0, lists[0], counts_dev[0], walk(0, 4), err, s)))
    }
    // 5 <= k <= 8 and k <= 4: several rows per MFMA tile
    if constexpr (X_LISTS) {
    is_x[8] = is_x[9] = true;
    ALS_TIMED_CLASS(T_SMALL8, 9, 8, (stb = launch_dual_small8_x(ctx, D, Y, Z, zb16, X->data, X->ld, r0, lists[9], counts_dev[9], walk(9, 8), LinvT, queue, err, s)))
    ALS_TIMED_CLASS(T_SMALL4, 8, 16, (stb = launch_dual_small4_x(ctx, D, Y, Z, zb16, X->data, X->ld, r0, lists[8], counts_dev[8], walk(8, 16), LinvT, queue + QUEUE_INTS, err, s)))
    } else {
    ALS_TIMED_CLASS(T_SMALL8, 9, 8, (launch_dual_small8(D, Y, Z, R, ldr, r0, lists[9], counts_dev[9], g, err, s)))
    ALS_TIMED_CLASS(T_SMALL4, 8, 16, (launch_dual_small4(D, Y, Z, R, ldr, r0, lists[8], counts_dev[8], g, err, s)))
    }
    }
    if constexpr (D >= 64) {
    // direct solver: short classes beyond k = 48 have no launch of their own (see wide_rest_limit)
    WideRest rest;
    int64_t room = wide_rest_limit(ctx->num_cu), joint = 0, beyond = 0;
    StepGrid wide[8];
    for (int c = 7; c >= 2; --c) {
        wide[c] = grid(c, 1);
        if (ws.cg || c == 2) continue;
        if (hints[c] >= 0 && hints[c] <= room) {
            room -= hints[c];
            joint += std::min<int64_t>(hints[c], caps[c]);
            wide[c].known = 0;
        } else {
            room = 0;
        }
        wide[c].rest = 0;
        rest.list[c - 3] = lists[c];
        rest.count[c - 3] = counts_dev[c];
        rest.known[c - 3] = (int32_t)wide[c].known;
        beyond += std::max<int64_t>(0, caps[c] - (int64_t)wide[c].known);
    }
#define ALS_WIDE(kt) \
    if (caps[kt - 1] > 0 && wide[kt - 1].known + wide[kt - 1].rest > 0 && stb == ALS_OK) { \
        timer_begin(ctx, T_DUAL_CLASS0 + kt - 1, s); \
        stb = launch_dual_wide##kt(ctx, D, Y, Z, zb16, R, ldr, r0, lists[kt - 1], counts_dev[kt - 1], wide[kt - 1], err, ws, s); \
        timer_end(ctx, s); \
    }
    if (!ws.cg) {
        ALS_TIMED_CLASS(T_DUAL_CLASS0 + 2, 2, 4, (launch_dual_triple(D, Y, Z, zb16, R, ldr, r0, lists[2], counts_dev[2], walk(2, 4), err, s)))
    } else {
        ALS_WIDE(3)
    }
    ALS_WIDE(4) ALS_WIDE(5) ALS_WIDE(6) ALS_WIDE(7) ALS_WIDE(8)
#undef ALS_WIDE
    if (!ws.cg && beyond > 0 && stb == ALS_OK) {
        timer_begin(ctx, D == 128 ? T_DUAL_CLASS0 + 7 : T_DUAL_CLASS0 + 3, s);
        stb = launch_dual_wide_rest(ctx, D, Y, Z, zb16, R, ldr, r0, rest,
                                    (unsigned)std::min<int64_t>(beyond, std::max<int64_t>(joint, 4 * ctx->num_cu)), err, s);
        timer_end(ctx, s);
    }
    }
    }
#undef ALS_TIMED_CLASS
    if (stb != ALS_OK) return stb;
    timer_begin(ctx, T_TRANSFORM_X, s);
    const unsigned xblocks = (unsigned)std::min<int64_t>(1024, std::max<int64_t>(1, (r1 - r0 + 127) / 128));
    if constexpr (X_LISTS) {
        using M = XMatrix<D, BF16>;
        typedef typename std::conditional<BF16, uint16_t, float>::type elem;
        XLists xl = {};
        int64_t tiles = 0;
        for (int c = 0; c < 10; ++c)
            if (caps[c] > 0 && !is_x[c]) {
                xl.list[xl.n] = lists[c];
                xl.count[xl.n++] = counts_dev[c];
                tiles += (caps[c] + 31) / 32;
            }
        for (int c = xl.n; c < 10; ++c) {
            xl.list[c] = xl.list[0];
            xl.count[c] = xl.count[0];
        }
        const TileGrid g = tile_grid(ctx->num_cu, tiles, r1 - r0, xl.n);
        auto launch = [&](auto threads) {
            constexpr int T = decltype(threads)::value;
            static const hipError_t attr_x = hipFuncSetAttribute((const void *)transform_lists_kernel<D, BF16, T>,
                                                                 hipFuncAttributeMaxDynamicSharedMemorySize, M::BYTES);  // once per process
            if (attr_x == hipSuccess)
                hipLaunchKernelGGL((transform_lists_kernel<D, BF16, T>), dim3(g.blocks), dim3(T), M::BYTES, s, (const float *)R, ldr,
                                   (elem *)X->data, X->ld, LinvT, r0, xl);
            return attr_x;
        };
        if (xl.n > 0) ALS_HIP(ctx, g.threads == 256 ? launch(std::integral_constant<int, 256>{}) : launch(std::integral_constant<int, 512>{}));
    } else {
        static const hipError_t attr_x = hipFuncSetAttribute((const void *)transform_kernel<D, false, BF16, false, false>,
                                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                                             (int)XfCfg<D>::LDS_BYTES);  // once per process
        ALS_HIP(ctx, attr_x);
        hipLaunchKernelGGL((transform_kernel<D, false, BF16, false, false>), dim3(xblocks), dim3(256), XfCfg<D>::LDS_BYTES, s,
                           (const void *)R, ldr, X->data, X->ld, LinvT, r0, r1, Y->indptr, (int64_t)dual_max, Gather{});
    }
    timer_end(ctx, s);
    ALS_HIP(ctx, hipGetLastError());
    return ALS_OK;
}

als_status launch_dual_prepare(als_ctx *ctx, const als_table *V, const float *G, const als_params *prm,
                               const als_csr *entries, int64_t r0, int64_t r1, bool factored, hipStream_t s) {
    const bool bf = V->dtype == ALS_BF16;
    switch (V->d) {
        case 16: return bf ? dual_prepare_typed<16, true>(ctx, V, G, prm, entries, r0, r1, factored, s) : dual_prepare_typed<16, false>(ctx, V, G, prm, entries, r0, r1, factored, s);
        case 32: return bf ? dual_prepare_typed<32, true>(ctx, V, G, prm, entries, r0, r1, factored, s) : dual_prepare_typed<32, false>(ctx, V, G, prm, entries, r0, r1, factored, s);
        case 64: return bf ? dual_prepare_typed<64, true>(ctx, V, G, prm, entries, r0, r1, factored, s) : dual_prepare_typed<64, false>(ctx, V, G, prm, entries, r0, r1, factored, s);
        case 128: return bf ? dual_prepare_typed<128, true>(ctx, V, G, prm, entries, r0, r1, factored, s) : dual_prepare_typed<128, false>(ctx, V, G, prm, entries, r0, r1, factored, s);
    }
    return fail(ctx, ALS_EDTYPE, "unsupported d");
}

als_status launch_dual_rows(als_ctx *ctx, const als_csr *Y, als_table *X, int64_t r0, int64_t r1, int dual_max,
                            const als_params *prm, const int32_t *const lists[10], const int32_t *const counts[10],
                            const int64_t caps[10], const int hints[10], hipStream_t s) {
    const bool bf = X->dtype == ALS_BF16;
    switch (X->d) {
        case 16: return bf ? dual_rows_typed<16, true>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s) : dual_rows_typed<16, false>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s);
        case 32: return bf ? dual_rows_typed<32, true>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s) : dual_rows_typed<32, false>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s);
        case 64: return bf ? dual_rows_typed<64, true>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s) : dual_rows_typed<64, false>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s);
        case 128: return bf ? dual_rows_typed<128, true>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s) : dual_rows_typed<128, false>(ctx, Y, X, r0, r1, dual_max, prm, lists, counts, caps, hints, s);
    }
    return fail(ctx, ALS_EDTYPE, "unsupported d");
}

}  // namespace als
