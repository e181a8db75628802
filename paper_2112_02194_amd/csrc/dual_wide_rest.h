// The lists of the classes 48 < k <= 128 as one launch sees them (dual_wide_rest.hip).
#pragma once

#include "als_internal.h"

namespace als {

struct WideRest {
    const int32_t *list[5], *count[5];  // class KT = 4 + i
    int32_t known[5];                   // rows that the launch of the class takes
};

als_status launch_dual_wide_rest(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                                 const WideRest &w, unsigned blocks, int32_t *err, hipStream_t s);

}  // namespace als
