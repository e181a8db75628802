// Row class 8 < k <= 16 (step: dual_rows_step.h).
#include "dual_rows_step.h"

namespace als {

template <int D>
__global__ __launch_bounds__(64) void dual_rows_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                       const float *__restrict__ values, const void *__restrict__ Z,
                                                       float *__restrict__ R, int64_t ldr, int64_t r0, const int32_t *__restrict__ list,
                                                       const int32_t *__restrict__ count_ptr, int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    walk_steps<RowsStep<D, false>>(indptr, indices, values, Z, R, ldr, r0, list, *count_ptr, err_flag, lds);
}

// bf16 Z, with X = R L^-1 taken along
template <int D>
__global__ __launch_bounds__(64) void dual_rows_x_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                         const float *__restrict__ values, const void *__restrict__ Z, XTable x,
                                                         int64_t r0, const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ count_ptr, int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    walk_steps_x<RowsStep<D, true>, D>(indptr, indices, values, Z, x, r0, list, *count_ptr, err_flag, lds);
}

template <int D>
static void launch_rows_typed(const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                              const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = RowsStep<D, false>::LDS_FLOATS * sizeof(float);
    static const int resident = resident_waves(dual_rows_kernel<D>, lds_bytes, w.num_cu);
    hipLaunchKernelGGL(dual_rows_kernel<D>, dim3(walk_blocks(resident, w.capacity, w.hint)), dim3(64), lds_bytes, s, Y->indptr,
                       Y->indices, Y->values, Z, R, ldr, r0, list, count_dev, err);
}
template <int D>
static void launch_rows_typed_x(const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list, const int32_t *count_dev,
                                WalkSize w, int32_t *err, hipStream_t s) {
    constexpr size_t lds_bytes = Parked<RowsStep<D, true>, D>::LDS_FLOATS * sizeof(float);
    static const int resident = resident_waves(dual_rows_x_kernel<D>, lds_bytes, w.num_cu);
    hipLaunchKernelGGL(dual_rows_x_kernel<D>, dim3(walk_blocks(resident, w.capacity, w.hint)), dim3(64), lds_bytes, s, Y->indptr,
                       Y->indices, Y->values, Z, x, r0, list, count_dev, err);
}

void launch_dual_k16(int d, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const int32_t *list,
                     const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
#define ALS_ROWS_CASE(dd) \
    case dd: launch_rows_typed<dd>(Y, Z, R, ldr, r0, list, count_dev, w, err, s); break;
    switch (d) { ALS_ROWS_CASE(16) ALS_ROWS_CASE(32) ALS_ROWS_CASE(64) ALS_ROWS_CASE(128) }
#undef ALS_ROWS_CASE
}
void launch_dual_k16_x(int d, const als_csr *Y, const void *Z, const XTable &x, int64_t r0, const int32_t *list,
                       const int32_t *count_dev, WalkSize w, int32_t *err, hipStream_t s) {
#define ALS_ROWS_CASE(dd) \
    case dd: launch_rows_typed_x<dd>(Y, Z, x, r0, list, count_dev, w, err, s); break;
    switch (d) { ALS_ROWS_CASE(32) ALS_ROWS_CASE(64) ALS_ROWS_CASE(128) }
#undef ALS_ROWS_CASE
}

}  // namespace als
