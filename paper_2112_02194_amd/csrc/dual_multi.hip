// Row class 16 < k <= 32 (step: dual_multi_step.h).
#include "dual_multi_step.h"

namespace als {

// LOOP = false: workgroup b takes step first_blk + b, if the list is that long (the launch for a list whose
// length the host knows from the previous call).  LOOP = true: grid-stride walk from first_blk to the end of
// the list, correct for any grid size (the length is only known on the device); the step inlined into a
// loop needs about twice the registers, so this form only serves what the first form did not cover.
template <int D, bool ZB, bool LOOP>
__global__ __launch_bounds__(64) void dual_multi_kernel(const int64_t *__restrict__ indptr,
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
        if (blk * 4 < count) dual_multi_step<D, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, blk, lds);
    } else {
        for (; blk * 4 < count; blk += gridDim.x) {
            dual_multi_step<D, ZB>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R), opaque(ldr),
                                  opaque(r0), opaque(list), opaque(count), opaque(err_flag), blk, opaque(lds));
            wave_sync();  // the next step reuses the LDS buffers
        }
    }
}

template <int D, bool ZB>
static void launch_multi_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                               const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = (multi_resident<ZB>() ? MultiCfg::LDS_FLOATS_RESIDENT : MultiCfg::LDS_FLOATS) * sizeof(float);
    if (g.known > 0)
        hipLaunchKernelGGL((dual_multi_kernel<D, ZB, false>), dim3(g.known), dim3(64), lds_bytes, s,
                           Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, 0, err);
    if (g.rest > 0)
        hipLaunchKernelGGL((dual_multi_kernel<D, ZB, true>), dim3(g.rest), dim3(64), lds_bytes, s,
                           Y->indptr, Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, (int)g.known, err);
}

void launch_dual_multi2(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                        const int32_t *list, const int32_t *count_dev, StepGrid g, int32_t *err, hipStream_t s) {
#define ALS_MULTI_CASE(dd)                                                                       \
    case dd:                                                                                     \
        if (zb16) launch_multi_typed<dd, true>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);    \
        else launch_multi_typed<dd, false>(Y, Z, R, ldr, r0, list, count_dev, g, err, s);        \
        break;
    switch (d) { ALS_MULTI_CASE(32) ALS_MULTI_CASE(64) ALS_MULTI_CASE(128) }  // the dual form stops at k = d
#undef ALS_MULTI_CASE
}

}  // namespace als
