// Steps of a list handed out to the wavefronts of a persistent launch.
#pragma once

#include "launch_size.h"

namespace als {

// A list's steps in eight contiguous parts, one per die (see xcd_step).  Each die's wavefronts (the launch has a multiple of
// eight workgroups) take the steps of its part in turn; where every wavefront gets many, they come from a counter per part instead, which is zero
// when the launch begins, a few at a time, and a wavefront whose part is used up goes on with the others, so that none is left with work
// while others have none.  The counters stand 64 bytes apart.
constexpr int QUEUE_PARTS = 8, QUEUE_STRIDE = 16, QUEUE_INTS = QUEUE_PARTS * QUEUE_STRIDE;

// All members are wavefront-uniform.
struct StepQueue {
    int32_t *counters;
    int steps, part, left, pos, end, stride;
    static constexpr int CHUNK = 4;
    constexpr int part_size() const { return list_steps(steps, QUEUE_PARTS); }
    constexpr int part_end(int p) const { return (p + 1) * part_size() < steps ? (p + 1) * part_size() : steps; }
    // look(counter) returns what the counter holds, take(counter, n) adds n to it and returns what it held
    template <class Look, class Take> constexpr int next(Look &&look, Take &&take) {  // a step, or -1 when there is none left
        while (pos >= end) {
            if (left == 0) return -1;
            const int first = part * part_size(), stop = part_end(part);
            int at = stop - first;  // may be negative
            if (at > 0 && (left == QUEUE_PARTS || look(counters + part * QUEUE_STRIDE) < at)) at = take(counters + part * QUEUE_STRIDE, CHUNK);
            if (at < stop - first) {
                pos = first + at;
                end = stop - pos < CHUNK ? stop : pos + CHUNK;
            } else {
                part = (part + 1) % QUEUE_PARTS;
                --left;
            }
        }
        const int step = pos;
        pos += stride;
        return step;
    }
};
// For wavefront `wave` of `per_block` of workgroup `block` of `blocks` (a multiple of eight).
constexpr StepQueue step_queue(int32_t *counters, int steps, int block, int blocks, int wave, int per_block) {
    StepQueue q{counters, steps, block % QUEUE_PARTS, QUEUE_PARTS, 0, 0, 1};
    if (steps < 64 * (int64_t)blocks * per_block) {
        q.left = 0;
        q.stride = blocks / QUEUE_PARTS * per_block;
        q.pos = q.part * q.part_size() + block / QUEUE_PARTS * per_block + wave;
        q.end = q.part_end(q.part);
    }
    return q;
}

}  // namespace als
