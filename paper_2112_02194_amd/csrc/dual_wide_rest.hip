// Rows of 48 < k <= 128 beyond those that the launches per class take (direct solver; step: dual_wide_step.h).
#include "dual_wide_rest.h"
#include "dual_wide_step.h"

namespace als {

// One launch for what is left of all classes, the longest rows first.  With launches of their own, short classes wait for a single row's
// chain of 15 to 30 us one after the other, and every class has one more launch that finds nothing where its hint was right (4 us
// each).  Which classes are short: wide_rest_limit.
// It takes the registers and the LDS of its largest class, at d = 128 one wavefront per SIMD (fp32) or two.
// What bounds it: the longest single row.
template <int D, bool ZB>
__global__ __launch_bounds__(64, 1) void dual_wide_rest_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                               const float *__restrict__ values, const void *__restrict__ Z,
                                                               float *__restrict__ R, int64_t ldr, int64_t r0, WideRest w,
                                                               int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    constexpr int LAST = D == 128 ? 4 : 0;  // list i: rows of class KT = 4 + i
    int64_t at = blockIdx.x;                // counted from the first row of list i that no other launch takes
    for (int i = LAST; i >= 0; --i) {
        const int64_t first = w.known[i], left = *w.count[i] - first;
        const int32_t *list = w.list[i];
        for (; at < left; at += gridDim.x) {
            const int item = (int)(first + at);
            auto step = [&](auto kt) {
                dual_wide_step<D, decltype(kt)::value, ZB, false>(opaque(indptr), opaque(indices), opaque(values), opaque(Z), opaque(R),
                                                                  opaque(ldr), opaque(r0), opaque(list), opaque(err_flag), item,
                                                                  opaque(lds), 0, 0.f);
            };
            switch (i) {  // uniform
                case 0: step(std::integral_constant<int, 4>{}); break;
                default:
                    if constexpr (D == 128) {
                        if (i == 1) step(std::integral_constant<int, 5>{});
                        else if (i == 2) step(std::integral_constant<int, 6>{});
                        else if (i == 3) step(std::integral_constant<int, 7>{});
                        else step(std::integral_constant<int, 8>{});
                    }
            }
            wave_sync();  // the next step reuses the LDS buffers
        }
        if (left > 0) at -= left;
    }
}

template <int D, bool ZB>
static als_status rest_typed(als_ctx *ctx, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const WideRest &w,
                             unsigned blocks, int32_t *err, hipStream_t s) {
    constexpr int lds_bytes = WideCfg<D, D == 128 ? 8 : 4>::LDS_FLOATS * (int)sizeof(float);
    static const hipError_t attr = hipFuncSetAttribute((const void *)dual_wide_rest_kernel<D, ZB>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);  // once per process
    ALS_HIP(ctx, attr);
    hipLaunchKernelGGL((dual_wide_rest_kernel<D, ZB>), dim3(blocks), dim3(64), lds_bytes, s, Y->indptr, Y->indices, Y->values, Z, R,
                       ldr, r0, w, err);
    return ALS_OK;
}

als_status launch_dual_wide_rest(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                                 const WideRest &w, unsigned blocks, int32_t *err, hipStream_t s) {
    if (d == 128) return zb16 ? rest_typed<128, true>(ctx, Y, Z, R, ldr, r0, w, blocks, err, s) : rest_typed<128, false>(ctx, Y, Z, R, ldr, r0, w, blocks, err, s);
    return zb16 ? rest_typed<64, true>(ctx, Y, Z, R, ldr, r0, w, blocks, err, s) : rest_typed<64, false>(ctx, Y, Z, R, ldr, r0, w, blocks, err, s);
}

}  // namespace als
