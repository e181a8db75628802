// Row class 8 < k <= 16 (step: dual_rows_step.h).
#include "dual_rows_step.h"

namespace als {

// The two launch forms of a step kernel (see StepGrid): one step per workgroup, or a grid-stride walk from
// step first_blk to the end of the list.
template <int D, bool ZB, bool LOOP>
__global__ __launch_bounds__(64) void dual_rows_kernel(const int64_t *__restrict__ indptr,
                                                       const int32_t *__restrict__ indices,
                                                       const float *__restrict__ values,
                                                       const void *__restrict__ Z, float *__restrict__ R,
                                                       int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                       const int32_t *__restrict__ count_ptr, int first_blk,
                                                       int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    const int count = *count_ptr;
    int blk = first_blk + blockIdx.x;
    if constexpr (!LOOP) {
        blk = xcd_step(blk, gridDim.x, (count + 3) / 4);
        if (blk * DualCfg<D>::RPW < count) dual_rows_step<D, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
    } else {
        for (; blk * DualCfg<D>::RPW < count; blk += gridDim.x) {
            dual_rows_step<D, ZB>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R), opaque(ldr), opaque(r0),
                              opaque(list), opaque(count), opaque(err_flag), blk, opaque(lds));
            wave_sync();  // the next step reuses the LDS buffers
        }
    }
}

template <int D, bool ZB>
static void launch_rows_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                              const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
    using C = DualCfg<D>;
    if (g.known > 0)
        hipLaunchKernelGGL((dual_rows_kernel<D, ZB, false>), dim3(g.known), dim3(64), C::LDS_FLOATS * sizeof(float), s,
                           Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, 0, err);
    if (g.rest > 0)
        hipLaunchKernelGGL((dual_rows_kernel<D, ZB, true>), dim3(g.rest), dim3(64), C::LDS_FLOATS * sizeof(float), s,
                           Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, (int)g.known, err);
}

void launch_dual_k16(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                     const int32_t *list, const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#define ALS_ROWS_CASE(dd)                                                                             \
    case dd:                                                                                          \
        if (zb16 && dd >= 32) launch_rows_typed<dd, (dd >= 32)>(Y, Z, R, ldr, r0, list, count_dev, g, err, s); \
        else launch_rows_typed<dd, false>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);              \
        break;
    switch (d) { ALS_ROWS_CASE(16) ALS_ROWS_CASE(32) ALS_ROWS_CASE(64) ALS_ROWS_CASE(128) }
#undef ALS_ROWS_CASE
}

}  // namespace als
