// Row classes k <= 4 and 5 <= k <= 8, compiled once each with -DSMALL_G=4 and -DSMALL_G=8 (step: dual_small_step.h).
#include "dual_small_step.h"

#ifndef SMALL_G
#error "compile with -DSMALL_G=8 or -DSMALL_G=4"
#endif

namespace als {

// The two launch forms of a step kernel (see StepGrid): one step per workgroup, or a grid-stride walk from
// step first_blk to the end of the list.
template <int D, int G, bool ZB, bool LOOP>
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
        if (blk < steps) dual_small_step<D, G, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
    } else {
        for (; blk < steps; blk += gridDim.x) {
            dual_small_step<D, G, ZB>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R), opaque(ldr), opaque(r0),
                              opaque(list), opaque(count), opaque(err_flag), blk, opaque(lds));
            wave_sync();  // the next step reuses the LDS buffers
        }
    }
}

template <int D, bool ZB>
static void launch_small_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                               const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
    using C = SmallCfg<D, SMALL_G>;
    if (g.known > 0)
        hipLaunchKernelGGL((dual_small_kernel<D, SMALL_G, ZB, false>), dim3(g.known), dim3(64),
                           C::LDS_FLOATS * sizeof(float), s, Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list,
                           count_dev, 0, err);
    if (g.rest > 0)
        hipLaunchKernelGGL((dual_small_kernel<D, SMALL_G, ZB, true>), dim3(g.rest), dim3(64),
                           C::LDS_FLOATS * sizeof(float), s, Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list,
                           count_dev, (int)g.known, err);
}

#if SMALL_G == 8
void launch_dual_small8(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                        const int32_t *list, const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#else
void launch_dual_small4(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                        const int32_t *list, const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#endif
#define ALS_SMALL_CASE(dd)                                                                              \
    case dd:                                                                                            \
        if (zb16 && dd >= 32) launch_small_typed<dd, (dd >= 32)>(Y, Z, R, ldr, r0, list, count_dev, g, err, s); \
        else launch_small_typed<dd, false>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);               \
        break;
    switch (d) { ALS_SMALL_CASE(16) ALS_SMALL_CASE(32) ALS_SMALL_CASE(64) ALS_SMALL_CASE(128) }
#undef ALS_SMALL_CASE
}

}  // namespace als
