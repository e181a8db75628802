// Row classes 48 < k <= 128, compiled once per class with -DWIDE_KT=4..8, and with -DWIDE_KT=3 all rows of up to 48 entries under conjugate
// gradients (step: dual_wide_step.h).
#include "dual_wide_step.h"

#ifndef WIDE_KT
#error "compile with -DWIDE_KT=3 .. 8"
#endif

namespace als {

// Direct solver: one row per workgroup (what no hint announced: dual_wide_rest.hip); conjugate gradients: a grid-stride walk over
// the list.
template <int D, int KT, bool ZB, bool CG>
__global__ __launch_bounds__(64, (CG || KT >= 7) ? 1 : (KT <= 4 ? 3 : 2)) void dual_wide_kernel(const int64_t *__restrict__ indptr,
                                                          const int32_t *__restrict__ indices,
                                                          const float *__restrict__ values,
                                                          const void *__restrict__ Z, float *__restrict__ R,
                                                          int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                          const int32_t *__restrict__ count_ptr,
                                                          int32_t *__restrict__ err_flag, int cg_iters, float cg_tol) {
    extern __shared__ float lds[];
    const int count = *count_ptr;
    int item = blockIdx.x;
    if constexpr (!CG) {
        item = xcd_step(item, gridDim.x, count);
        if (item < count)
            dual_wide_step<D, KT, ZB, CG>(indptr, indices, values, Z, R, ldr, r0, list, err_flag, item, lds, cg_iters, cg_tol);
    } else {
        for (; item < count; item += gridDim.x) {
            dual_wide_step<D, KT, ZB, CG>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R),
                                          opaque(ldr), opaque(r0), opaque(list), opaque(err_flag), item, opaque(lds),
                                          opaque(cg_iters), opaque(cg_tol));
            wave_sync();  // the next step reuses the LDS buffers
        }
    }
}

#define ALS_WIDE_NAME2(kt) launch_dual_wide##kt
#define ALS_WIDE_NAME(kt) ALS_WIDE_NAME2(kt)

template <int D, bool ZB>
static als_status wide_typed(als_ctx *ctx, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0,
                             const int32_t *list, const int32_t *count_dev, StepGrid g, int32_t *err, const WideSolver &ws,
                             hipStream_t s) {
    using C = WideCfg<D, WIDE_KT>;
    constexpr int lds_bytes = (int)(C::LDS_FLOATS * sizeof(float));
    auto launch = [&](auto kern, unsigned blocks) {
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(64), lds_bytes, s, Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list, count_dev,
                           err, ws.iters, ws.tol);
    };
    if (ws.cg) {  // one launch covers the list
        static const hipError_t attr_cg = hipFuncSetAttribute((const void *)dual_wide_kernel<D, WIDE_KT, ZB, true>,
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);  // once per process
        ALS_HIP(ctx, attr_cg);
        launch(dual_wide_kernel<D, WIDE_KT, ZB, true>, g.known + g.rest);
    } else if constexpr (WIDE_KT > 3) {
        static const hipError_t attr = hipFuncSetAttribute((const void *)dual_wide_kernel<D, WIDE_KT, ZB, false>,
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);  // once per process
        ALS_HIP(ctx, attr);
        launch(dual_wide_kernel<D, WIDE_KT, ZB, false>, g.known);
    }
    return ALS_OK;
}

als_status ALS_WIDE_NAME(WIDE_KT)(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr,
                                  int64_t r0, const int32_t *list, const int32_t *count_dev, StepGrid g,
                                  int32_t *err, const WideSolver &ws, hipStream_t s) {
    if (g.known + (ws.cg ? g.rest : 0u) == 0) return ALS_OK;
    if (d == 128)
        return zb16 ? wide_typed<128, true>(ctx, Y, Z, R, ldr, r0, list, count_dev, g, err, ws, s)
                    : wide_typed<128, false>(ctx, Y, Z, R, ldr, r0, list, count_dev, g, err, ws, s);
    if constexpr (WIDE_KT <= 4) {  // the dual form reaches k <= 64 at d = 64
        if (d == 64)
            return zb16 ? wide_typed<64, true>(ctx, Y, Z, R, ldr, r0, list, count_dev, g, err, ws, s)
                        : wide_typed<64, false>(ctx, Y, Z, R, ldr, r0, list, count_dev, g, err, ws, s);
    }
    return fail(ctx, ALS_EDTYPE, "wide dual kernel: unsupported d");
}

}  // namespace als
