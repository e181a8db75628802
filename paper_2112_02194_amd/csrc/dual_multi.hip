// Row class 16 < k <= 32 (step: dual_multi_step.h).
#include "dual_multi_step.h"

namespace als {

template <int D>
__global__ __launch_bounds__(64) void dual_multi_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                       const float *__restrict__ values, const void *__restrict__ Z,
                                                       float *__restrict__ R, int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                       const int32_t *__restrict__ count_ptr, int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    walk_steps<MultiStep<D, false>>(indptr, indices, values, Z, R, ldr, r0, list, *count_ptr, err_flag, lds);
}

// bf16 Z, with X = R L^-1 taken along
template <int D>
__global__ __launch_bounds__(64, D == 128 ? 2 : 3) void dual_multi_x_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                         const float *__restrict__ values, const void *__restrict__ Z, XTable x,
                                                         int64_t r0, const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ count_ptr, int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    walk_steps_x<MultiStep<D, true>, D>(indptr, indices, values, Z, x, r0, list, *count_ptr, err_flag, lds);
}

template <int D>
static void launch_multi_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                              const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = MultiStep<D, false>::LDS_FLOATS * sizeof(float);
    static const int resident = resident_waves(dual_multi_kernel<D>, lds_bytes, w.num_cu);
    hipLaunchKernelGGL(dual_multi_kernel<D>, dim3(walk_blocks(resident, w.capacity, w.hint)), dim3(64), lds_bytes, s, Y->indptr,
                       Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, err);
}
template <int D>
static void launch_multi_typed_x(const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list, const int32_t *count_dev,
                                WalkSize w, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = Parked<MultiStep<D, true>, D>::LDS_FLOATS * sizeof(float);
    static const int resident = resident_waves(dual_multi_x_kernel<D>, lds_bytes, w.num_cu);
    hipLaunchKernelGGL(dual_multi_x_kernel<D>, dim3(walk_blocks(resident, w.capacity, w.hint)), dim3(64), lds_bytes, s, Y->indptr,
                       Y->indices, Y->values, Z, x, r0, list, count_dev, err);
}

void launch_dual_multi2(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                     const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
#define ALS_ROWS_CASE(dd) \
    case dd: launch_multi_typed<dd>(Y, Z, R, ldr, r0, list, count_dev, w, err, s); break;
    switch (d) { ALS_ROWS_CASE(32) ALS_ROWS_CASE(64) ALS_ROWS_CASE(128) }  // the dual form stops at k = d
#undef ALS_ROWS_CASE
}
void launch_dual_multi2_x(int d, const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list,
                       const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
#define ALS_ROWS_CASE(dd) \
    case dd: launch_multi_typed_x<dd>(Y, Z, x, r0, list, count_dev, w, err, s); break;
    switch (d) { ALS_ROWS_CASE(32) ALS_ROWS_CASE(64) ALS_ROWS_CASE(128) }
#undef ALS_ROWS_CASE
}

}  // namespace als
