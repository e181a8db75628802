// The class lists of a call as one launch sees them (dual_few.hip).
#pragma once

#include "als_internal.h"

namespace als {

// rows per step of lists 0..9 (see dual_few.hip)
constexpr int FEW_ROWS[10] = {4, 4, 1, 1, 1, 1, 1, 1, 16, 8};
// Steps that all lists together can hold at most for the common launch.  Fold-ins against 1M items (d = 128, fp32), a
// launch per class / one launch, us: 256 rows 170 / 101, 6000 rows 268 / 169, 20 000 rows 372 / 284, 60 000 rows
// 652 / 581 (about 131 000 steps), 150 000 rows 854 / 963.  Just below the line at the other sizes (55 000 rows): d = 16 110 / 94,
// d = 32 155 / 131, d = 64 286 / 236, bf16 111 / 94, 137 / 115, 201 / 159 and (d = 128) 418 / 369; epochs of 12 000 to
// 34 000 rows gain 5 to 40 %.
constexpr int64_t FEW_STEPS = 1 << 17;

// Rows of 33 to 48 entries (d >= 64) that an earlier call saw, or that there can be, from which on they have the launch that takes
// four of them per wavefront, the same operations on each.  Calls with rows of 40 entries only, in the common launch / their own, us:
// d = 64 2500 rows 69 / 76, 5000 88 / 86, 40 000 231 / 207 (bf16: 2500 63 / 67, 30 000 172 / 140); d = 128 2500 rows 129 / 129, 5000 179 / 167
// (bf16: 2500 106 / 100, 5000 134 / 117).
constexpr int64_t few_triple_rows(int d) { return d == 64 ? 16384 : 4096; }

struct FewLists {
    const int32_t *list[10], *count[10];
    int32_t start[11];  // first workgroup of each list; the last: the number of workgroups
};

als_status launch_dual_few(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                           const FewLists &few, int32_t *err, hipStream_t s);

}  // namespace als
