// How many queries of a top-k call are worked on together (host arithmetic only, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace als {

constexpr int TOPK_SELECT_THREADS = 256;  // the select kernel's workgroup; one per query, and a launch holds fewer than 2^32 threads
constexpr int TOPK_MIN_BATCH = 64;        // queries of one workgroup of the bound and of the scan kernel

// Batches of about equal size whose `per_query` bytes fit `limit` bytes, in whole groups of `group` queries (the last batch
// may be smaller).
inline int64_t topk_batch(int64_t queries, int64_t per_query, int64_t group, int64_t limit) {
    const int64_t launch_max = (int64_t)0xffffffff / TOPK_SELECT_THREADS;
    const int64_t fit = std::max(group, std::min(limit / std::max<int64_t>(per_query, 1), launch_max) / group * group);
    const int64_t batches = (queries + fit - 1) / fit;
    return std::min(queries, ((queries + batches - 1) / batches + group - 1) / group * group);
}

// The next batch to try where the workspace for this one cannot be allocated; the same one where there is none.
inline int64_t topk_smaller_batch(int64_t batch) {
    return batch <= TOPK_MIN_BATCH ? batch : std::max<int64_t>(TOPK_MIN_BATCH, batch / 2 / TOPK_MIN_BATCH * TOPK_MIN_BATCH);
}

}  // namespace als
