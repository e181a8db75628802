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

// Rows of 33 to 48 entries (d >= 64) that an earlier call saw from which on they have the launch that takes four of them per wavefront,
// the same operations on each.  (What a list can hold says little: 15 000 rows of 1 to 128 entries that no call had seen, d = 64, bf16, took
// 174 us in the common launch and 184 with the class, 1900 rows, in a launch sized for 15 000.)  In the common launch / their own, us a
// call; rows of 40 entries:
//   d = 64, fp32   8000 87 / 84, 10 000 106 / 105, 13 000 117 / 119, 16 000 128 / 124, 20 000 142 / 147, 30 000 176 / 177: no clear line
//   d = 64, bf16   4000 59 / 65, 6000 67 / 66, 8000 74 / 69, 16 000 114 / 101
//   d = 128, fp32  3000 122 / 123, 4000 140 / 136, 8000 198 / 174       d = 128, bf16  2000 83 / 82, 3000 97 / 91, 6000 130 / 110
// and among others (rows of 20 to 60 entries, 39 in 100 of them in the class): d = 64, bf16 5900 112 / 115, 7800 128 / 125, fp32 5900
// 132 / 136, 11 700 189 / 194; d = 128, fp32 3100 198 / 199, 3900 234 / 230, bf16 1600 108 / 113, 2300 126 / 126, 3100 145 / 138.
constexpr int64_t few_triple_rows(int d, bool zb16) { return d == 64 ? (zb16 ? 6144 : 16384) : (zb16 ? 2304 : 3584); }

struct FewLists {
    const int32_t *list[10], *count[10];
    int32_t start[11];  // first workgroup of each list; the last: the number of workgroups
};

als_status launch_dual_few(als_ctx *ctx, int d, const als_csr *Y, const void *Z, bool zb16, float *R, int64_t ldr, int64_t r0,
                           const FewLists &few, int32_t *err, hipStream_t s);

}  // namespace als
