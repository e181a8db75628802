// All dual row classes in one launch, for calls whose class lists are short: a launch per class leaves the chip to a few
// workgroups at a time and waits for the slowest of each class in turn.  Workgroup b works on step b - start[c] of the class c
// with start[c] <= b < start[c + 1]; a list's length is read on the device, steps beyond it return at once.
// What bounds it: the longest single step (a row of up to 128 entries solved by one wavefront).  The kernel takes the
// registers and the LDS of its largest class, which long lists pay for: see FEW_STEPS.
#include "dual_few.h"
#include "dual_multi_step.h"
#include "dual_rows_step.h"
#include "dual_small_step.h"
#include "dual_triple_step.h"
#include "dual_wide_step.h"

namespace als {

// 16 < k <= 32 keeps the tiles of its four rows in registers in the launch of its own.  This kernel takes the registers and LDS of its
// largest class, and with fp32 Z those tiles took it from 87 to 166 registers at d = 32 and from 105 to 240 at d = 64, for all classes:
// 300k rows of 3 entries (d = 32) 115 -> 122 us, 40k rows of 40 / 56 entries (d = 64) 221 / 303 -> 244 / 325 us.  With a second gather
// and one chunk of the tiles under way, 122 registers either way: 113 and 205 / 282 us; 40k rows of 25 entries 76 -> 76 us (d = 32) and
// 120 -> 124 us (d = 64), the price.
template <bool ZB> constexpr bool few_keeps_tiles() { return ZB; }

template <int D, bool ZB> constexpr int few_lds_floats() {
    int n = RowsCfg<D, ZB>::LDS_FLOATS;
    auto take = [&](int x) { n = x > n ? x : n; };
    take(SmallCfg<D, 4>::LDS_FLOATS);
    take(SmallCfg<D, 8>::LDS_FLOATS);
    if constexpr (D >= 32) take(MultiCfg<D, ZB, few_keeps_tiles<ZB>()>::LDS_FLOATS);
    if constexpr (D >= 64) take(TripleCfg<D, ZB, 1>::LDS_FLOATS);
    if constexpr (D == 64) take(WideCfg<D, 4>::LDS_FLOATS);
    if constexpr (D == 128) take(WideCfg<D, 8>::LDS_FLOATS);
    return n;
}

template <int D, bool ZB>
__global__ __launch_bounds__(64) void dual_few_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                      const float *__restrict__ values, const void *__restrict__ Z,
                                                      float *__restrict__ R, int64_t ldr, int64_t r0, FewLists few,
                                                      int32_t *__restrict__ err_flag) {
    extern __shared__ float lds[];
    const int b = blockIdx.x;
    int c = 0;
    while (c < 9 && b >= few.start[c + 1]) ++c;
    const int step = b - few.start[c], count = *few.count[c];
    const int32_t *list = few.list[c];
    // lists 0..7: ceil(k / 16) - 1, lists 8 and 9: k <= 4 and 5 <= k <= 8
    if (step >= list_steps(count, FEW_ROWS[c])) return;
    auto wide = [&](auto kt) {
        constexpr int KT = decltype(kt)::value;
        if constexpr (16 * KT <= (D == 128 ? 128 : 64) && D >= 64)
            dual_wide_step<D, KT, ZB, false>(indptr, indices, values, Z, R, ldr, r0, list, err_flag, step, lds, 0, 0.f);
    };
    switch (c) {  // uniform
        case 0: dual_rows_step<D, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, step, lds); break;
        case 1:
            if constexpr (D >= 32) dual_multi_step<D, ZB, few_keeps_tiles<ZB>()>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, step, lds);
            break;
        case 2:
            if constexpr (D >= 64) dual_triple_row<D, ZB>(indptr, indices, values, Z, R, ldr, r0, list, err_flag, step, lds);
            break;
        case 3: wide(std::integral_constant<int, 4>{}); break;
        case 4: wide(std::integral_constant<int, 5>{}); break;
        case 5: wide(std::integral_constant<int, 6>{}); break;
        case 6: wide(std::integral_constant<int, 7>{}); break;
        case 7: wide(std::integral_constant<int, 8>{}); break;
        case 8: dual_small_step<D, 4, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, step, lds); break;
        case 9: dual_small_step<D, 8, ZB>(indptr, indices, values, Z, R, ldr, r0, list, count, err_flag, step, lds); break;
    }
}

template <int D, bool ZB>
static als_status few_typed(als_ctx *ctx, const als_csr *Y, const void *Z, float *R, int64_t ldr, int64_t r0, const FewLists &few,
                            int32_t *err, hipStream_t s) {
    constexpr int lds_bytes = few_lds_floats<D, ZB>() * (int)sizeof(float);
    static const hipError_t attr = hipFuncSetAttribute((const void *)dual_few_kernel<D, ZB>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);  // once per process
    ALS_HIP(ctx, attr);
    hipLaunchKernelGGL((dual_few_kernel<D, ZB>), dim3(few.start[10]), dim3(64), lds_bytes, s, Y->indptr, Y->indices, Y->values, Z, R,
                       ldr, r0, few, err);
    return ALS_OK;
}

als_status launch_dual_few(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                           const FewLists &few, int32_t *err, hipStream_t s) {
    switch (d) {
        case 16: return few_typed<16, false>(ctx, Y, Z, R, ldr, r0, few, err, s);
        case 32: return zb16 ? few_typed<32, true>(ctx, Y, Z, R, ldr, r0, few, err, s) : few_typed<32, false>(ctx, Y, Z, R, ldr, r0, few, err, s);
        case 64: return zb16 ? few_typed<64, true>(ctx, Y, Z, R, ldr, r0, few, err, s) : few_typed<64, false>(ctx, Y, Z, R, ldr, r0, few, err, s);
        case 128: return zb16 ? few_typed<128, true>(ctx, Y, Z, R, ldr, r0, few, err, s) : few_typed<128, false>(ctx, Y, Z, R, ldr, r0, few, err, s);
    }
    return fail(ctx, ALS_EDTYPE, "unsupported d");
}

}  // namespace als
