// Primal row update: the d x d normal equations of the paper's Eq. 4, formed and solved per row
// exactly in the order of Algorithm 1 lines 4-10:
//     A = alpha*G + lambda*I ;  b = 0
//     for every stored (u, i, y):  A += v_i (x) v_i ;  b += y * v_i
//     x_u = A^{-1} b            (Cholesky, A is symmetric positive definite because lambda > 0)
//
// One workgroup owns one row (or one segment of a long row).  d < 64: the gathered rows of the fixed
// table go straight from global memory into MFMA operand registers (no staging): lane (m, kk)
// loads the NC consecutive columns NC*m.. of the kk-th entry of the current step, wavefront I of
// the workgroup accumulates tile-row I of V_I^T V_I (see Geo<>).  d >= 64: accumulate_staged.  The finished
// tiles are written to LDS together with alpha*G + lambda*I, factorised there, and the two triangular solves
// give the new row, which is rounded once to the table's element type.
//
// Rows longer than `split` are cut into segments (the counterpart of the paper's Section 4.3 row
// splitting): each segment's partial statistics go to a workspace and a second kernel sums them
// in a fixed order before the same factorisation.
#include <type_traits>

#include "dual_common.h"
#include "tri_solve.h"

namespace als {

template <int D> struct Team {
    static constexpr int WAVES = Geo<D>::NC;      // one wavefront per tile-row
    static constexpr int THREADS = 64 * WAVES;
    static_assert(THREADS == primal_threads(D), "the launch sizes count on it");
    static constexpr int LD = D + 1;              // LDS leading dimension (odd: conflict-free both ways)
    static constexpr size_t LDS_BYTES = (size_t)(D * LD + 6 * D + 8) * sizeof(float);
};

// ---------------------------------------------------------------------------------------------- accumulate
// Accumulates, for entries [begin, end) of the CSR arrays, tile-row `I` of sum v (x) v into acc[]
// and, in the wavefront of tile-row 0 only, this lane's share of sum y*v into bsum[] (lane (m,kk) holds
// columns NC*m.. of entries kk mod KS).
template <int D, bool BF16>
__device__ __forceinline__ void accumulate_entries(const void *__restrict__ V, int64_t ld,
                                                   const int32_t *__restrict__ indices,
                                                   const float *__restrict__ values, int64_t begin, int64_t end,
                                                   int I, typename AccT<Geo<D>::ACC>::type (&acc)[Geo<D>::NC],
                                                   float (&bsum)[Geo<D>::NC]) {
    using G = Geo<D>;
    constexpr int NC = G::NC, TM = G::TM, KS = G::KS, U = 8;
    const int lane = opaque_tid() & 63;
    const int m = lane % TM, kk = lane / TM;
    const uint32_t ld32 = (uint32_t)ld;  // the leading dimension fits 32 bits (checked on the host)
    const bool first_row = __builtin_amdgcn_readfirstlane(I) == 0;
    for (int64_t base = begin; base < end; base += 64) {
        const int64_t p = base + lane;
        const int myidx = p < end ? indices[p] : -1;
        const float myy = p < end ? (values ? values[p] : 1.f) : 0.f;
        const int cnt = (int)((end - base) < 64 ? (end - base) : 64);
        const int nsteps = (cnt + KS - 1) / KS;
        for (int s0 = 0; s0 < nsteps; s0 += U) {
            // all lane exchanges of the batch first, then all loads: one wait instead of one per load
            int idx[U];
            float x[U][NC], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = (s0 + u) * KS + kk;
                idx[u] = __shfl(myidx, e & 63);
                y[u] = __shfl(myy, e & 63);
            }
            if ((s0 + U) * KS <= cnt) {  // uniform: every slot of the batch holds an entry
#pragma unroll
                for (int u = 0; u < U; ++u)
                    load_vec<NC, BF16>(V, (int64_t)((uint64_t)(uint32_t)idx[u] * ld32) + NC * m, x[u]);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool have = (s0 + u) * KS + kk < cnt;
                    y[u] = have ? y[u] : 0.f;
                    if (have) {
                        load_vec<NC, BF16>(V, (int64_t)((uint64_t)(uint32_t)idx[u] * ld32) + NC * m, x[u]);
                    } else {
#pragma unroll
                        for (int c = 0; c < NC; ++c) x[u][c] = 0.f;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float a = x[u][0];
#pragma unroll
                for (int c = 1; c < NC; ++c) a = (I == c) ? x[u][c] : a;
#pragma unroll
                for (int j = 0; j < NC; ++j) acc[j] = mfma<D>(a, x[u][j], acc[j]);
            }
            if (first_row) {  // scalar branch: only the wavefront of tile-row 0 carries the right-hand side
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int j = 0; j < NC; ++j) bsum[j] += y[u] * x[u][j];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- accumulate, d >= 64
// The same statistics for d = 64 or 128 on the bf16 matrix cores.  bf16 entries are operands as they are; fp32 entries are
// cut into three bf16 parts, x = h + m + l exactly, and a product is taken as hh' + hm' + mh' + hl' + lh' + mm' (what is
// dropped is below the rounding of an fp32 product); the products of 16 entries are summed inside the matrix core from
// zero, small terms first, and join the running sum by a vector addition, which rounds to nearest.
//
// Batches of 32 entries: the workgroup gathers each row once (16 bytes of the parts per thread, whole rows side by side, the
// next batch requested before this one's products), cuts it and leaves the parts in LDS.  The product contracts over the
// entries, so an operand needs eight entries of one column per lane, which is what the transposing LDS read delivers
// (ds_read_b64_tr_b16: of four rows of 16 elements, lane i of a group of 16 gets column i).  The 64-byte blocks of a row
// are permuted by its number, so that the four rows of a read lie in different banks.  Wavefront w owns the block pairs
// p with p % 4 == w of the upper block triangle (ten at d = 128, three at d = 64).
// On return acc[p / 4] holds pair p = (gi, gj): element v of lane (m, kq) is entry
// (32 gi + 8 (v / 4) + 4 kq + v % 4, 32 gj + m), and thread c < D holds b[c] in b.
//
// What bounds it: with fp32 tables the matrix cores (480 products of 32 clocks per batch and d = 128, four wavefronts; the
// fp32 instruction, which has no use for the symmetry either, takes 4.3 times as long), with bf16 tables the gather and the
// solve that follows.  Together with the solve by four wavefronts, against a gather by every wavefront, the fp32 instruction
// and one solving wavefront: 825 000 rows of 129 to 512 entries, bf16, 59 -> 34 ms; the segments of a 10M x 10M fp32 half
// 7.6 -> 3.45 ms, its rows of 129 to 512 entries 2.66 -> 1.44 ms (all d = 128).
template <int D> struct BlockPairs {
    static constexpr int NB = D / 32, COUNT = NB * (NB + 1) / 2, PER_WAVE = (COUNT + 3) / 4;
    static constexpr int first(int p) {  // pairs in the order (0,0) (0,1) .. (0,NB-1) (1,1) ..
        int g = 0;
        while (p >= NB - g) {
            p -= NB - g;
            ++g;
        }
        return g;
    }
    static constexpr int second(int p) {
        int g = 0;
        while (p >= NB - g) {
            p -= NB - g;
            ++g;
        }
        return g + p;
    }
};

template <int D, bool BF16> struct Staging {
    static constexpr int BATCH = 32, PARTS = BF16 ? 1 : 3, ROW = 2 * D, PLANE = BATCH * ROW;
    static constexpr int BUFS = BF16 ? 2 : 1;  // two buffers need one barrier per batch, one needs two; three parts take the space
    static constexpr int PPR = D / 8, EPP = 256 / PPR, NP = BATCH / EPP;  // pieces of 8 columns per row; entries per pass; passes
    static constexpr int BYTES = BUFS * PARTS * PLANE, SUM_BYTES = EPP * D * 4;  // the sums of b reuse the space
    static constexpr int LDS_BYTES = BYTES > SUM_BYTES ? BYTES : SUM_BYTES;
    // rows that share 256 bytes of LDS lie in different banks anyway; the next ones get their blocks exchanged
    static __device__ int block_shift(int entry) { return (entry / (256 / ROW)) % (ROW / 64); }
};

template <int D, bool BF16>
__device__ __forceinline__ void accumulate_staged(const void *__restrict__ V, int64_t ld, const int32_t *__restrict__ indices,
                                                  const float *__restrict__ values, int64_t begin, int64_t end, int wave_s,
                                                  char *lds, floatx16 (&acc)[BlockPairs<D>::PER_WAVE], float &b) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef short shortx4 __attribute__((ext_vector_type(4)));
    typedef short shortx8 __attribute__((ext_vector_type(8)));
    using S = Staging<D, BF16>;
    using BP = BlockPairs<D>;
    const int tid = opaque_tid(), lane = tid & 63;
    const uint32_t ld32 = (uint32_t)ld;  // the leading dimension fits 32 bits (checked on the host)
    const int pc = tid % S::PPR, e0 = tid / S::PPR;  // this thread's piece, its entry of a pass
    constexpr int RAW = BF16 ? 1 : 2;                // 16-byte loads per piece

    float4 raw[S::NP][RAW];
    float y[S::NP], bsum[8];
    int32_t idx[S::NP];
#pragma unroll
    for (int c = 0; c < 8; ++c) bsum[c] = 0.f;
    auto ids = [&](int64_t base) {
#pragma unroll
        for (int i = 0; i < S::NP; ++i) {
            const int64_t p = base + i * S::EPP + e0;
            idx[i] = p < end ? indices[p] : -1;
        }
    };
    auto fetch = [&](int64_t base) {
#pragma unroll
        for (int i = 0; i < S::NP; ++i) {
#pragma unroll
            for (int r = 0; r < RAW; ++r) raw[i][r] = make_float4(0.f, 0.f, 0.f, 0.f);
            y[i] = 0.f;
            if (idx[i] >= 0) {
                const int64_t off = (int64_t)((uint64_t)(uint32_t)idx[i] * ld32) + 8 * pc;
                y[i] = values ? values[base + i * S::EPP + e0] : 1.f;
                if constexpr (BF16) {
                    raw[i][0] = *(const float4 *)((const uint16_t *)V + off);
                } else {
                    raw[i][0] = *(const float4 *)((const float *)V + off);
                    raw[i][1] = *(const float4 *)((const float *)V + off + 4);
                }
            }
        }
    };
    auto stash = [&](char *buf) {
#pragma unroll
        for (int i = 0; i < S::NP; ++i) {
            const int e = i * S::EPP + e0;
            char *dst = buf + e * S::ROW + (((pc / 4) ^ S::block_shift(e)) * 64 + (pc % 4) * 16);
            float x[8];
            if constexpr (BF16) {
                *(float4 *)dst = raw[i][0];
                const u32x4 w = __builtin_bit_cast(u32x4, raw[i][0]);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    x[2 * c] = __uint_as_float(w[c] << 16);
                    x[2 * c + 1] = __uint_as_float(w[c] & 0xffff0000u);
                }
            } else {
                x[0] = raw[i][0].x; x[1] = raw[i][0].y; x[2] = raw[i][0].z; x[3] = raw[i][0].w;
                x[4] = raw[i][RAW - 1].x; x[5] = raw[i][RAW - 1].y; x[6] = raw[i][RAW - 1].z; x[7] = raw[i][RAW - 1].w;
                float r[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) r[c] = x[c];
#pragma unroll
                for (int part = 0; part < 3; ++part) {
                    *(u32x4 *)(dst + part * S::PLANE) = u32x4{pack_upper(r[0], r[1]), pack_upper(r[2], r[3]), pack_upper(r[4], r[5]), pack_upper(r[6], r[7])};
#pragma unroll
                    for (int c = 0; c < 8; ++c) r[c] = lower_part(r[c]);
                }
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) bsum[c] = fmaf(y[i], x[c], bsum[c]);
        }
    };
    // this lane's address inside a plane for column block 0, entries 0..: row 8 (lane / 32) + lane % 16 / 4, columns
    // 16 (lane / 16 % 2) + 4 (lane % 4) ..; the block number enters by exclusive or
    const int trow = 8 * (lane >> 5) + ((lane >> 2) & 3);
    const int tbase = trow * S::ROW + S::block_shift(trow) * 64 + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    auto operand = [&](const char *plane, int ks, int g) {  // eight entries of column 32 g + lane % 32
        typedef __attribute__((address_space(3))) shortx4 *lds_ptr;
        const char *at = plane + (tbase ^ (g * 64)) + 16 * ks * S::ROW;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 4 * S::ROW));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    ids(begin);
    fetch(begin);
    ids(begin + S::BATCH);
    int which = 0;
    for (int64_t base = begin; base < end; base += S::BATCH) {
        char *buf = lds + which * (S::PARTS * S::PLANE);
        stash(buf);
        fetch(base + S::BATCH);  // past the end: zeros, no loads
        ids(base + 2 * S::BATCH);
        __syncthreads();
        static_for<0, BP::COUNT>([&](auto pp) {
            constexpr int pr = decltype(pp)::value, gi = BP::first(pr), gj = BP::second(pr);
            if (wave_s == pr % 4) {  // scalar branch
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 A[S::PARTS], B[S::PARTS];
#pragma unroll
                    for (int t = 0; t < S::PARTS; ++t) {
                        A[t] = operand(buf + t * S::PLANE, ks, gi);
                        B[t] = gi == gj ? A[t] : operand(buf + t * S::PLANE, ks, gj);
                    }
                    if constexpr (BF16) {
                        acc[pr / 4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0], B[0], acc[pr / 4], 0, 0, 0);
                    } else {
                        constexpr int PA[6] = {1, 2, 0, 1, 0, 0}, PB[6] = {1, 0, 2, 0, 1, 0};  // mm lh hl mh hm hh
                        floatx16 t16;
#pragma unroll
                        for (int v = 0; v < 16; ++v) t16[v] = 0.f;
#pragma unroll
                        for (int t = 0; t < 6; ++t) t16 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[PA[t] % S::PARTS], B[PB[t] % S::PARTS], t16, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[pr / 4][v] += t16[v];
                    }
                }
            }
        });
        if constexpr (S::BUFS == 1) __syncthreads();
        else which ^= 1;
    }
    // b: the threads of one piece, summed in a fixed order
    if constexpr (S::BUFS == 2) __syncthreads();
    float *sums = (float *)lds;
    *(float4 *)(sums + e0 * D + 8 * pc) = make_float4(bsum[0], bsum[1], bsum[2], bsum[3]);
    *(float4 *)(sums + e0 * D + 8 * pc + 4) = make_float4(bsum[4], bsum[5], bsum[6], bsum[7]);
    __syncthreads();
    b = 0.f;
    if (tid < D) {
#pragma unroll 8
        for (int e = 0; e < S::EPP; ++e) b += sums[e * D + tid];
    }
    __syncthreads();  // the caller may overwrite the LDS
}

// Sum bsum over the KS lanes that hold the same columns; afterwards lanes with kk == 0 hold b.
template <int D> __device__ __forceinline__ void fold_b(float (&bsum)[Geo<D>::NC]) {
    constexpr int TM = Geo<D>::TM, KS = Geo<D>::KS, NC = Geo<D>::NC;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int off = TM * KS / 2; off >= TM; off >>= 1) bsum[c] += __shfl_xor(bsum[c], off);
    }
}

// ---------------------------------------------------------------------------------------------- direct solve
// LDS layout of the direct solver: lower triangle, the solver's auxiliary and result
// buffers (tri_solve.h), the right-hand side.
template <int D> struct Packed {
    static constexpr int TRI = tri_row<D>(D);
    static constexpr int OFF_COL = TRI;                        // the solver's auxiliary buffer
    static constexpr int OFF_T = OFF_COL + TRI_AUX_FLOATS<D>;     // tbuf[D]
    static constexpr int OFF_RHS = OFF_T + D;      // rhs[D]
    static constexpr size_t LDS_BYTES = (size_t)(OFF_RHS + D) * sizeof(float);
};

// Called by the whole workgroup behind a barrier: solves the packed system and stores the row, rounded once to the
// table's element type.  Returns at once in the wavefronts that have nothing left to do; wavefront 0 stores.  One or two
// panels (d < 64) are worked on by wavefront 0 alone; a Cholesky factorisation in LDS with two barriers per column
// took an epoch of 50k x 30k rows (d = 32, half of them longer than 32) to 838 us instead of 444.  It divided by
// square roots; the panels' reciprocals are the hardware's after one Newton step, and the error against fp64 was no larger for
// it.  With block_solve it is (rows of 1 to 500 entries, lambda 1e-4 to 1, against rows in lanes as in tri_solve)
// d = 16 2.16e-7 -> 2.00e-7, d = 32 2.54e-7 -> 2.20e-7 on average.  It takes inverses of diagonal blocks, which pays at the weights
// of Eq. 3 in use and costs where a row's system is nearly singular (rows of 1 to 300 entries, d = 16, error relative to tri_solve's:
// alpha = 0.05 0.91, 1e-4 0.97, 1e-5 1.06, 1e-6 with lambda = 1e-4 1.13; d = 32 0.82, 0.93, 0.99, 1.04).
template <int D, bool BF16>
__device__ __forceinline__ void packed_solve_store(float *lds, void *X, int64_t xoff, int wave_s, int32_t *err_flag) {
    const int lane = opaque_tid() & 63;
    float *tbuf = lds + Packed<D>::OFF_T, *aux = lds + Packed<D>::OFF_COL, *rhs = lds + Packed<D>::OFF_RHS;
    int k = D;
    asm volatile("" : "+s"(k));  // opaque on purpose: with a compile-time step count the steps merge into one block,
                                 // whose scheduling runs out of registers
    if constexpr (D >= 64) {
        team_tri_eliminate<D>(lds, aux, rhs, wave_s, err_flag);
        if (wave_s != 0) return;
        tri_back<D>(lds, tbuf, rhs[lane], D > 64 ? rhs[64 + lane] : 0.f, aux[lane], D > 64 ? aux[64 + lane] : 1.f, k);
    } else {
        if (wave_s != 0) return;
        block_solve<D>(lds, aux, tbuf, lane < D ? rhs[lane] : 0.f, k, err_flag);
    }
    for (int c = lane; c < D; c += 64) store_elem<BF16>(X, xoff + c, tbuf[c]);
}

// Four consecutive entries of G, whose base need not be 16-byte aligned (`aligned`: it is; uniform for the launch).
__device__ __forceinline__ float4 load_g4(const float *__restrict__ G, int at, bool aligned) {
    if (aligned) return *(const float4 *)(G + at);
    return make_float4(G[at], G[at + 1], G[at + 2], G[at + 3]);
}

// ---------------------------------------------------------------------------------------------- conjugate gradients
template <int D>
__device__ __forceinline__ float block_dot(float v, float *red /* [THREADS/64] */) {
    const int lane = opaque_tid() & 63, w = opaque_tid() >> 6;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();  // red is free again
    if (lane == 0) red[w] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < Team<D>::THREADS / 64; ++i) s += red[i];
    return s;
}

template <int D>
__device__ __forceinline__ void cg_solve_lds(const float *a, float *aux, int max_iters, float tol) {
    constexpr int LD = Team<D>::LD;
    float *rvec = aux, *pvec = aux + D, *xvec = aux + 2 * D, *bvec = aux + 3 * D, *red = aux + 4 * D;
    const int i = opaque_tid();
    const bool mine = i < D;
    auto matvec = [&](const float *v) {  // row i of A times v (A symmetric: read column i, contiguous in LDS)
        float s = 0.f;
        if (mine) {
#pragma unroll 8
            for (int j = 0; j < D; ++j) s += a[j * LD + i] * v[j];
        }
        return s;
    };
    float x = mine ? xvec[i] : 0.f;
    const float b = mine ? bvec[i] : 0.f;
    float r = b - matvec(xvec);
    float pv = r;
    const float bb = block_dot<D>(b * b, red);
    float rs = block_dot<D>(r * r, red);
    const float stop = fmaxf(tol * tol * bb, CG_RESIDUAL_FLOOR);
    for (int it = 0; it < max_iters && rs > stop; ++it) {
        __syncthreads();
        if (mine) pvec[i] = pv;
        __syncthreads();
        const float ap = matvec(pvec);
        const float pap = block_dot<D>(pv * ap, red);
        if (!(pap > 0.f)) break;  // only when the numbers have left the fp32 range; the same in every thread
        const float alpha = rs / pap;
        x += alpha * pv;
        r -= alpha * ap;
        const float rs_new = block_dot<D>(r * r, red);
        pv = r + (rs_new / rs) * pv;
        rs = rs_new;
    }
    (void)rvec;
    __syncthreads();
    if (mine) xvec[i] = x;
    __syncthreads();
}

// ---------------------------------------------------------------------------------------------- kernels
enum PrimalMode { MODE_FUSED = 0, MODE_SEGMENT = 1 };

// One work item.  `last`: the workgroup has no further item, so the wavefronts that do not solve may retire
// as soon as their tiles are in LDS (their SIMD slots go to the next workgroup).  Returns false when the
// calling wavefront has retired.
template <int D, bool BF16, int MODE>
__device__ __forceinline__ bool primal_step(
    const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices, const float *__restrict__ values,
    const void *__restrict__ V, int64_t ldv, const float *__restrict__ G, float alpha, float lambda,
    void *__restrict__ X, int64_t ldx, int64_t row_begin, const int32_t *__restrict__ row_list,
    const Segment *__restrict__ segs, float *__restrict__ partials, int32_t *__restrict__ err_flag, int solver,
    int cg_iters, float cg_tol, int64_t item, bool last, float *lds) {
    using GE = Geo<D>;
    constexpr int NC = GE::NC, TM = GE::TM, ACC = GE::ACC, LD = Team<D>::LD;
    typedef typename AccT<ACC>::type acc_t;
    float *a = lds, *aux = lds + D * LD, *bvec = aux + 3 * D;

    const int lane = opaque_tid() & 63, wave = opaque_tid() >> 6;
    const int m = lane % TM, kk = lane / TM;
    int64_t u = 0, begin, end;
    if constexpr (MODE == MODE_FUSED) {
        u = row_begin + row_list[item];
        begin = indptr[u];
        end = indptr[u + 1];
    } else {
        begin = segs[item].begin;
        end = segs[item].end;
    }

    if constexpr (D >= 64) {
        using BP = BlockPairs<D>;
        const int wave_s = __builtin_amdgcn_readfirstlane(wave);
        floatx16 acc[BP::PER_WAVE];
        float b;
#pragma unroll
        for (int j = 0; j < BP::PER_WAVE; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
        accumulate_staged<D, BF16>(V, ldv, indices, values, begin, end, wave_s, (char *)lds, acc, b);
        // put4(r, c, values) for columns c .. c + 3 of row r: the blocks of the lower block triangle, whole
        auto deliver = [&](auto &&put4) {
            const int m32 = lane & 31, kq = lane >> 5;
            static_for<0, BP::COUNT>([&](auto pp) {
                constexpr int pr = decltype(pp)::value, gi = BP::first(pr), gj = BP::second(pr);
                if (wave_s == pr % 4) {
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        put4(32 * gj + m32, 32 * gi + 8 * x + 4 * kq,
                             make_float4(acc[pr / 4][4 * x], acc[pr / 4][4 * x + 1], acc[pr / 4][4 * x + 2], acc[pr / 4][4 * x + 3]));
                }
            });
        };
        if constexpr (MODE == MODE_SEGMENT) {  // only the lower block triangle of the partial is written and read
            float *out = partials + item * (int64_t)(D * D + D);
            deliver([&](int r, int c, const float4 &v) { *(float4 *)(out + r * D + c) = v; });
            if (opaque_tid() < D) out[D * D + opaque_tid()] = b;
            (void)last;
            return true;
        } else {
            const bool g_aligned = ((uintptr_t)G & 15) == 0;
            auto finished = [&](int r, int c, const float4 &v) {  // + alpha*G + lambda*I
                const float4 g = load_g4(G, r * D + c, g_aligned);
                return make_float4(v.x + alpha * g.x + (r == c ? lambda : 0.f), v.y + alpha * g.y + (r == c + 1 ? lambda : 0.f),
                                   v.z + alpha * g.z + (r == c + 2 ? lambda : 0.f), v.w + alpha * g.w + (r == c + 3 ? lambda : 0.f));
            };
            if (solver == ALS_SOLVER_DIRECT) {  // uniform for the launch
                // lower triangle of A = alpha*G + lambda*I + V_I^T V_I, packed: what a row holds beyond its last tile of
                // 16 columns is not stored
                deliver([&](int r, int c, const float4 &v) {
                    if (c < 16 * (r / 16 + 1)) *(float4 *)(lds + tri_row<D>(r) + c) = finished(r, c, v);
                });
                if (opaque_tid() < D) lds[Packed<D>::OFF_RHS + opaque_tid()] = b;
                __syncthreads();
                packed_solve_store<D, BF16>(lds, X, u * ldx, wave_s, err_flag);
                if (last && wave_s != 0) return false;
            } else {
                // entry (r, c) at a[c*LD + r], both triangles; warm start from the row's current content
                deliver([&](int r, int c, const float4 &v) {
                    const float4 w = finished(r, c, v);
                    const float e[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (c + i <= r) a[(c + i) * LD + r] = a[r * LD + c + i] = e[i];
                });
                if (opaque_tid() < D) bvec[opaque_tid()] = b;
                for (int c = opaque_tid(); c < D; c += Team<D>::THREADS) aux[2 * D + c] = load_elem<BF16>(X, u * ldx + c);
                __syncthreads();
                cg_solve_lds<D>(a, aux, cg_iters, cg_tol);
                for (int c = opaque_tid(); c < D; c += Team<D>::THREADS) store_elem<BF16>(X, u * ldx + c, aux[2 * D + c]);
            }
            if (!last) __syncthreads();  // the solver is done with the LDS before the next row arrives
            return true;
        }
    } else {
        acc_t acc[NC];
        float bsum[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            bsum[j] = 0.f;
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[j][v] = 0.f;
        }
        accumulate_entries<D, BF16>(V, ldv, indices, values, begin, end, wave, acc, bsum);
        fold_b<D>(bsum);
        auto deliver = [&](auto &&put, auto &&put_b) {
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int v = 0; v < ACC; ++v) put(NC * acc_row<D>(v, lane) + wave, NC * m + j, acc[j][v]);
            if (wave == 0 && kk == 0) {
#pragma unroll
                for (int j = 0; j < NC; ++j) put_b(NC * m + j, bsum[j]);
            }
        };
        if constexpr (MODE == MODE_SEGMENT) {
            float *out = partials + item * (int64_t)(D * D + D);
            deliver([&](int r, int c, float v) { out[r * D + c] = v; }, [&](int c, float v) { out[D * D + c] = v; });
            (void)last;
            return true;
        } else {
            if (solver == ALS_SOLVER_DIRECT) {  // uniform for the launch
                deliver([&](int r, int c, float v) { if (c <= r) lds[tri_row<D>(r) + c] = v + alpha * G[r * D + c] + (r == c ? lambda : 0.f); },
                        [&](int c, float v) { lds[Packed<D>::OFF_RHS + c] = v; });
                __syncthreads();
                const int wave_s = __builtin_amdgcn_readfirstlane(wave);
                packed_solve_store<D, BF16>(lds, X, u * ldx, wave_s, err_flag);
                if (last && wave_s != 0) return false;
            } else {
                // entry (r,c) at a[c*LD + r]; warm start from the row's current content
                deliver([&](int r, int c, float v) { a[c * LD + r] = v + alpha * G[r * D + c] + (r == c ? lambda : 0.f); },
                        [&](int c, float v) { bvec[c] = v; });
                for (int c = opaque_tid(); c < D; c += Team<D>::THREADS) aux[2 * D + c] = load_elem<BF16>(X, u * ldx + c);
                __syncthreads();
                cg_solve_lds<D>(a, aux, cg_iters, cg_tol);
                for (int c = opaque_tid(); c < D; c += Team<D>::THREADS) store_elem<BF16>(X, u * ldx + c, aux[2 * D + c]);
            }
            if (!last) __syncthreads();  // before the next row's tiles overwrite the LDS
            return true;
        }
    }
}

// What the workgroups of a primal kernel share.
struct PrimalArgs {
    const int64_t *indptr;
    const int32_t *indices;
    const float *values;
    const void *V;
    int64_t ldv;
    const float *G;
    float alpha, lambda;
    void *X;
    int64_t ldx, row_begin;
    const int32_t *row_list, *row_count;  // MODE_FUSED: work item = the whole row u = row_begin + row_list[item]
    const Segment *segs;                  // MODE_SEGMENT: segment `item`; raw partial statistics are written to
    const int32_t *seg_count;             // partials[item][D*D + D] (row-major D x D, then b)
    float *partials;
    int32_t *err_flag;
    int solver, cg_iters;
    float cg_tol;
};

// Workgroup `b` of `blocks` of the items from `first` on.  The two launch forms (see StepGrid): LOOP = false, item first + b if
// there is one; LOOP = true, grid-stride walk.
template <int D, bool BF16, int MODE, bool LOOP>
__device__ __forceinline__ void primal_items(const PrimalArgs &p, int first, int b, int blocks, float *lds) {
    const int64_t nitems = MODE == MODE_FUSED ? *p.row_count : *p.seg_count;
    int64_t item = (int64_t)first + b;
    if constexpr (!LOOP) {
        if (item < nitems)
            primal_step<D, BF16, MODE>(p.indptr, p.indices, p.values, p.V, p.ldv, p.G, p.alpha, p.lambda, p.X, p.ldx, p.row_begin, p.row_list,
                                       p.segs, p.partials, p.err_flag, p.solver, p.cg_iters, p.cg_tol, item, true, lds);
    } else {
        for (; item < nitems; item += blocks) {
            const bool last = item + blocks >= nitems;
            if (!primal_step<D, BF16, MODE>(opaque(p.indptr), opaque(p.indices), opaque(p.values), opaque(p.V), opaque(p.ldv), opaque(p.G),
                                            opaque(p.alpha), opaque(p.lambda), opaque(p.X), opaque(p.ldx), opaque(p.row_begin),
                                            opaque(p.row_list), opaque(p.segs), opaque(p.partials), opaque(p.err_flag), opaque(p.solver),
                                            opaque(p.cg_iters), opaque(p.cg_tol), item, last, opaque(lds)))
                return;
        }
    }
}

template <int D, bool BF16, int MODE>
__global__ __launch_bounds__(Team<D>::THREADS, D < 64 ? 2 : (D == 128 && !BF16 ? 3 : 4)) void primal_kernel(PrimalArgs p) {
    extern __shared__ float lds[];
    primal_items<D, BF16, MODE, false>(p, 0, blockIdx.x, gridDim.x, lds);
}
// Segments (the first `seg_blocks` workgroups) and whole rows in one launch: neither waits for the other's last ones.  The segments' workgroups
// take the LDS of the solver too, so for d >= 64 only where all find a place at a time.  Epoch of 2000 x 1500 (d = 16)
// 103 -> 90 us, of 50k x 30k (d = 32) 315 -> 300 us (150 us of rows and 25 of segments before), 256 rows folded in (d = 128) 81.9 -> 80.8 us.
template <int D, bool BF16, bool LOOP>
__global__ __launch_bounds__(Team<D>::THREADS, D < 64 ? (LOOP ? 1 : 2) : (D == 128 && !BF16 ? (LOOP ? 2 : 3) : 4 - LOOP)) void primal_both_kernel(
    PrimalArgs p, int first_seg, int seg_blocks, int first_row) {
    extern __shared__ float lds[];
    const int b = blockIdx.x;
    if (b < seg_blocks) primal_items<D, BF16, MODE_SEGMENT, LOOP>(p, first_seg, b, seg_blocks, lds);
    else primal_items<D, BF16, MODE_FUSED, LOOP>(p, first_row, b - seg_blocks, (int)gridDim.x - seg_blocks, lds);
}

// One element of a long row's partials, summed in a fixed order.
template <int D> __device__ __forceinline__ float segment_sum(const float *p0, int nseg) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    int g = 0;
    for (; g + 4 <= nseg; g += 4) {
        s0 += p0[(int64_t)(g + 0) * (D * D + D)];
        s1 += p0[(int64_t)(g + 1) * (D * D + D)];
        s2 += p0[(int64_t)(g + 2) * (D * D + D)];
        s3 += p0[(int64_t)(g + 3) * (D * D + D)];
    }
    for (; g < nseg; ++g) s0 += p0[(int64_t)g * (D * D + D)];
    return (s0 + s1) + (s2 + s3);
}

// Adds the segment partials of every long row in a fixed order: workgroup (x, y) handles elements
// [256y, 256y+256) of long row x and overwrites the row's first partial with the sum.
template <int D>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const LongRow *__restrict__ long_rows,
                                                              float *__restrict__ partials,
                                                              const int32_t *__restrict__ n_long_ptr) {
    const int n_long = *n_long_ptr;
    for (int row = blockIdx.x; row < n_long; row += gridDim.x) {
    const LongRow lr = long_rows[row];
    const int e = blockIdx.y * 256 + opaque_tid();
    if (e >= D * D + D || lr.nseg <= 1) continue;
    if (D >= 64 && e < D * D && e % D / 32 > e / D / 32) continue;  // segments leave the lower block triangle only
    float *p0 = partials + (int64_t)lr.seg_first * (D * D + D) + e;
    p0[0] = segment_sum<D>(p0, lr.nseg);
    }
}

// Below d = 64 a row's partials are a few kilobytes each: the solving workgroup sums them itself, and
// reduce_partials_kernel is not launched.
template <int D> constexpr bool sums_segments() { return D < 64; }

// Loads the summed statistics of one long row, adds alpha*G + lambda*I, solves, stores.  `last` and the
// return value as in primal_step.
template <int D, bool BF16>
__device__ __forceinline__ bool reduce_solve_step(const LongRow lr, const float *__restrict__ partials,
                                                  const float *__restrict__ G, float alpha, float lambda,
                                                  void *__restrict__ X, int64_t ldx, int32_t *__restrict__ err_flag,
                                                  int solver, int cg_iters, float cg_tol, bool last, float *lds) {
    constexpr int LD = Team<D>::LD, T = Team<D>::THREADS;
    float *a = lds, *aux = lds + D * LD, *bvec = aux + 3 * D;
    const float *p0 = partials + (int64_t)lr.seg_first * (D * D + D);
    const int nsum = sums_segments<D>() ? lr.nseg : 1;
    if (solver == ALS_SOLVER_DIRECT) {
        const bool g_aligned = ((uintptr_t)G & 15) == 0;
        for (int e = opaque_tid(); e < D * D / 4; e += T) {
            const int r = e / (D / 4), c = 4 * (e % (D / 4));
            if (c < 16 * (r / 16 + 1)) {
                const float4 v = nsum > 1 ? make_float4(segment_sum<D>(p0 + 4 * e, nsum), segment_sum<D>(p0 + 4 * e + 1, nsum),
                                                        segment_sum<D>(p0 + 4 * e + 2, nsum), segment_sum<D>(p0 + 4 * e + 3, nsum))
                                          : *(const float4 *)(p0 + 4 * e);
                const float4 g = load_g4(G, 4 * e, g_aligned);
                *(float4 *)(lds + tri_row<D>(r) + c) =
                    make_float4(v.x + alpha * g.x + (r == c ? lambda : 0.f), v.y + alpha * g.y + (r == c + 1 ? lambda : 0.f),
                                v.z + alpha * g.z + (r == c + 2 ? lambda : 0.f), v.w + alpha * g.w + (r == c + 3 ? lambda : 0.f));
            }
        }
        if (opaque_tid() < D) lds[Packed<D>::OFF_RHS + opaque_tid()] = segment_sum<D>(p0 + D * D + opaque_tid(), nsum);
        __syncthreads();
        const int wave_s = __builtin_amdgcn_readfirstlane(opaque_tid() >> 6);
        packed_solve_store<D, BF16>(lds, X, lr.row * ldx, wave_s, err_flag);
        if (last && wave_s != 0) return false;
        if (!last) __syncthreads();
        return true;
    }
    for (int e = opaque_tid(); e < D * D + D; e += T) {
        const float s = segment_sum<D>(p0 + e, nsum);
        if (e < D * D) {
            const int r = e / D, c = e % D;
            if (D >= 64 && c > r) continue;  // the lower triangle serves both
            const float v = s + alpha * G[e] + (r == c ? lambda : 0.f);
            a[c * LD + r] = v;
            if (D >= 64) a[r * LD + c] = v;
        } else {
            bvec[e - D * D] = s;
        }
    }
    for (int c = opaque_tid(); c < D; c += T) aux[2 * D + c] = load_elem<BF16>(X, lr.row * ldx + c);
    __syncthreads();
    cg_solve_lds<D>(a, aux, cg_iters, cg_tol);
    const float *xout = aux + 2 * D;
    for (int c = opaque_tid(); c < D; c += T) store_elem<BF16>(X, lr.row * ldx + c, xout[c]);
    if (!last) __syncthreads();
    return true;
}

// The two launch forms (see StepGrid): LOOP = false, long row first + blockIdx.x if there is one; LOOP = true, from `first` on in strides of
// the grid.  The direct solver takes the walk for all rows (it costs eight registers there; a launch of its own for the rows that no hint
// announced was one more that mostly found nothing), conjugate gradients both: their loop takes longer in the walk (15 000 rows of 700
// entries, bf16, the kernel in one form / in two: d = 64 383 / 370 us, d = 128 2.79 / 2.72 ms).
template <int D, bool BF16, bool LOOP>
__global__ __launch_bounds__(Team<D>::THREADS) void reduce_solve_kernel(
    const LongRow *__restrict__ long_rows, const float *__restrict__ partials, const float *__restrict__ G,
    float alpha, float lambda, void *__restrict__ X, int64_t ldx, const int32_t *__restrict__ n_long_ptr, int first,
    int32_t *__restrict__ err_flag, int solver, int cg_iters, float cg_tol) {
    extern __shared__ float lds[];
    const int n_long = *n_long_ptr;
    int row = first + (int)blockIdx.x;
    if constexpr (!LOOP) {
        if (row < n_long)
            reduce_solve_step<D, BF16>(long_rows[row], partials, G, alpha, lambda, X, ldx, err_flag, solver, cg_iters, cg_tol, true, lds);
    } else {
        for (; row < n_long; row += gridDim.x) {
            const bool last = row + (int)gridDim.x >= n_long;
            if (!reduce_solve_step<D, BF16>(long_rows[row], opaque(partials), opaque(G), opaque(alpha), opaque(lambda),
                                            opaque(X), opaque(ldx), opaque(err_flag), opaque(solver), opaque(cg_iters),
                                            opaque(cg_tol), last, opaque(lds)))
                return;
        }
    }
}

// ---------------------------------------------------------------------------------------------- launchers
// LDS of a workgroup that accumulates (segments), solves (summed segments), or does both
template <int D, bool BF16> static constexpr size_t staging_lds_bytes() {
    if constexpr (D >= 64) return Staging<D, BF16>::LDS_BYTES;
    else return 0;
}
template <int D> static size_t solve_lds_bytes(int solver) {
    return solver == ALS_SOLVER_DIRECT ? Packed<D>::LDS_BYTES : Team<D>::LDS_BYTES;
}

// counters[0] = number of long rows, counters[1] = number of their segments (device memory); row_list: rows solved whole.
template <int D, bool BF16>
static als_status primal_typed(als_ctx *ctx, const als_csr *Y, const als_table *V, const float *G, const als_params *prm, als_table *X,
                               int64_t r0, const LongRow *long_rows, const Segment *segs, const int32_t *counters, int64_t seg_capacity,
                               StepGrid g_long, StepGrid g_seg, const int32_t *row_list, const int32_t *row_count, StepGrid g_row, hipStream_t s) {
    const bool any_long = g_seg.known + g_seg.rest > 0;
    if (any_long) {
        als_status st = ensure(ctx, ctx->seg_partials, (size_t)seg_capacity * (D * D + D) * sizeof(float));
        if (st != ALS_OK) return st;
    }
    int32_t *err = (int32_t *)((char *)ctx->small.p + SM_COUNTERS) + 2;
    const int cg_iters = prm->cg_max_iters > 0 ? prm->cg_max_iters : 2 * D;
    const float cg_tol = prm->cg_tol > 0.f ? prm->cg_tol : 1e-6f;
    float *partials = (float *)ctx->seg_partials.p;
    const PrimalArgs args = {Y->indptr, Y->indices, Y->values, V->data, V->ld, G, prm->alpha, prm->lambda, X->data, X->ld, r0, row_list,
                             row_count, segs, counters + 1, partials, err, prm->solver, cg_iters, cg_tol};
    constexpr int T = Team<D>::THREADS;
    constexpr size_t seg_lds = staging_lds_bytes<D, BF16>();  // at most 24 KB: no attribute needed
    const size_t solve_lds = solve_lds_bytes<D>(prm->solver), row_lds = std::max(solve_lds, seg_lds);
#define ALS_LDS(kern)                                                                                                               \
    {                                                                                                                               \
        static const hipError_t attr = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,          \
                                                           (int)Team<D>::LDS_BYTES); /* once per process */                         \
        ALS_HIP(ctx, attr);                                                                                                         \
    }
    auto both = primal_both_kernel<D, BF16, false>, both_loop = primal_both_kernel<D, BF16, true>;
    ALS_LDS(both_loop)
    auto walk = [&] {  // rows and segments that no hint announced
        if (g_seg.rest + g_row.rest > 0)
            hipLaunchKernelGGL(both_loop, dim3(g_seg.rest + g_row.rest), dim3(T), row_lds, s, args, (int)g_seg.known, (int)g_seg.rest,
                               (int)g_row.known);
    };
    const bool together = D < 64 || (int64_t)g_seg.known + g_row.known <= 4 * ctx->num_cu;
    if (together) {
        ALS_LDS(both)
        timer_begin(ctx, T_PRIMAL, s);
        if (g_seg.known + g_row.known > 0)
            hipLaunchKernelGGL(both, dim3(g_seg.known + g_row.known), dim3(T), row_lds, s, args, 0, (int)g_seg.known, 0);
        walk();
        timer_end(ctx, s);
    } else if constexpr (D >= 64) {
        timer_begin(ctx, T_SEGMENT, s);
        if (g_seg.known > 0)
            hipLaunchKernelGGL((primal_kernel<D, BF16, MODE_SEGMENT>), dim3(g_seg.known), dim3(T), seg_lds, s, args);
        if (g_seg.rest > 0) walk();
        timer_end(ctx, s);
    }
    if (any_long) {
        timer_begin(ctx, T_REDUCE, s);
        const unsigned red_blocks = std::max(1u, g_long.known + g_long.rest);  // grid-stride over the long rows
        if constexpr (!sums_segments<D>())
            hipLaunchKernelGGL(reduce_partials_kernel<D>, dim3(red_blocks, (D * D + D + 255) / 256), dim3(256), 0, s, long_rows, partials, counters);
        auto kred = reduce_solve_kernel<D, BF16, false>, kred_loop = reduce_solve_kernel<D, BF16, true>;
        ALS_LDS(kred)
        ALS_LDS(kred_loop)
        auto reduce = [&](auto kern, unsigned blocks, unsigned first) {
            if (blocks > 0)
                hipLaunchKernelGGL(kern, dim3(blocks), dim3(T), solve_lds, s, long_rows, (const float *)partials, G, prm->alpha, prm->lambda, X->data,
                                   X->ld, counters, (int)first, err, prm->solver, cg_iters, cg_tol);
        };
        if (prm->solver == ALS_SOLVER_DIRECT) {
            reduce(kred_loop, red_blocks, 0);
        } else {
            reduce(kred, g_long.known, 0);
            reduce(kred_loop, g_long.rest, g_long.known);
        }
        timer_end(ctx, s);
    }
    // Rows of their own launch come last: between the segments and their sums they made calls of 15 000 rows of 100 to 300 entries
    // (d = 64, fp32) 3 % slower, 371 -> 382 us.
    if constexpr (D >= 64) {
        if (!together) {
            auto rows = primal_kernel<D, BF16, MODE_FUSED>;
            ALS_LDS(rows)
            timer_begin(ctx, T_PRIMAL, s);
            if (g_row.known > 0) hipLaunchKernelGGL(rows, dim3(g_row.known), dim3(T), row_lds, s, args);
            if (g_seg.rest == 0) walk();
            timer_end(ctx, s);
        }
    }
#undef ALS_LDS
    ALS_HIP(ctx, hipGetLastError());
    return ALS_OK;
}

#define ALS_DISPATCH(fn, d, bf, ...)                                                       \
    switch (d) {                                                                           \
        case 16: return bf ? fn<16, true>(__VA_ARGS__) : fn<16, false>(__VA_ARGS__);       \
        case 32: return bf ? fn<32, true>(__VA_ARGS__) : fn<32, false>(__VA_ARGS__);       \
        case 64: return bf ? fn<64, true>(__VA_ARGS__) : fn<64, false>(__VA_ARGS__);       \
        case 128: return bf ? fn<128, true>(__VA_ARGS__) : fn<128, false>(__VA_ARGS__);    \
    }                                                                                      \
    return fail(ctx, ALS_EDTYPE, "unsupported d")

als_status launch_primal(als_ctx *ctx, const als_csr *Y, const als_table *V, const float *G, const als_params *prm, als_table *X,
                         int64_t r0, const LongRow *long_rows, const Segment *segs, const int32_t *counters, int64_t seg_capacity,
                         StepGrid g_long, StepGrid g_seg, const int32_t *row_list, const int32_t *row_count, StepGrid g_row, hipStream_t s) {
    const bool bf = V->dtype == ALS_BF16;
    ALS_DISPATCH(primal_typed, V->d, bf, ctx, Y, V, G, prm, X, r0, long_rows, segs, counters, seg_capacity, g_long, g_seg, row_list, row_count, g_row, s);
}

}  // namespace als
