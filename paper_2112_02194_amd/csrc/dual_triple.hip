// Row class 32 < k <= 48, direct solver (step: dual_triple_step.h).
#include "dual_triple_step.h"

namespace als {

template <int D, bool ZB>
__global__ __launch_bounds__(64, 2) void dual_triple_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                            const float *__restrict__ values, const void *__restrict__ Z,
                                                            float *__restrict__ R, int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                            const int32_t *__restrict__ count_ptr, int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    walk_steps<TripleStep<D, ZB, 4>>(indptr, indices, values, Z, R, ldr, r0, list, *count_ptr, err_flag, lds);
}

template <int D, bool ZB>
static void launch_triple_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                                const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = TripleStep<D, ZB, 4>::LDS_FLOATS * sizeof(float);
    static const int resident = resident_waves(dual_triple_kernel<D, ZB>, lds_bytes, w.num_cu);
    hipLaunchKernelGGL((dual_triple_kernel<D, ZB>), dim3(walk_blocks(resident, w.capacity, w.hint)), dim3(64), lds_bytes, s, Y->indptr,
                       Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, err);
}

void launch_dual_triple(int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                        const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
    if (d == 128) {
        if (zb16) launch_triple_typed<128, true>(Y, Z, R, ldr, r0, list, count_dev, w, err, s);
        else launch_triple_typed<128, false>(Y, Z, R, ldr, r0, list, count_dev, w, err, s);
    } else {
        if (zb16) launch_triple_typed<64, true>(Y, Z, R, ldr, r0, list, count_dev, w, err, s);
        else launch_triple_typed<64, false>(Y, Z, R, ldr, r0, list, count_dev, w, err, s);
    }
}

}  // namespace als
