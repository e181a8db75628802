// How many workgroups a row list gets (host arithmetic only, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace als {

// How a list of `capacity` steps at most is launched when its length is only known on the device.  The
// row kernels come in two forms: one step per workgroup (launched with `known` workgroups, the length the
// previous call on the same matrix saw; steps beyond the true length return at once), and a grid-stride walk
// over everything from step `known` on (launched with `rest` workgroups; finds nothing to do when the hint
// was right).  Together they cover the list whatever the hint was.  (Rows of 9 to 48 entries have one form, which walks: walk_blocks;
// those of 49 to 128 share one launch for the rest, dual_wide_rest.hip.)
struct StepGrid {
    unsigned known, rest;
};

// hint: the list's length as an earlier call saw it, or -1.  A workgroup that finds nothing to do costs 0.2 ns of the
// launch.  A list that can hold a few thousand steps only is launched whole: one launch instead of two (an epoch of
// 2000 x 1500: 184 -> 170 us).  Without a hint, too, the list is covered in the one-step form as far as it can reach or
// `blind_limit` allows: the grid-stride form takes a quarter to a third longer per step (1M x 1M, d = 64, no hint:
// 7.3 -> 6.5 ms).  A launch holds fewer than 2^32 threads, so the limit depends on the kernel's workgroup: with one limit of
// 2^24 workgroups for all, the 2.2e7 steps of 16 < k <= 32 of a 100M-row epoch (64 threads each) took the grid-stride form
// from there on, and 256 threads were too many.  One launch may take both parts together, or the first
// part with the `beside` workgroups of another list.
inline StepGrid step_grid(int num_cu, int threads, int64_t capacity, int64_t hint, int per_cu, int64_t blind_limit,
                          int64_t beside = 0) {
    StepGrid g = {0u, 0u};
    if (capacity <= 0) return g;
    constexpr int64_t WHOLE = 4096;
    const int64_t walkers = (int64_t)num_cu * per_cu;
    const int64_t launch_max = (int64_t)0xffffffff / threads - walkers - beside;
    const int64_t wanted = capacity <= WHOLE ? capacity : (hint < 0 ? blind_limit : hint);
    g.known = (unsigned)std::min(wanted, std::min(capacity, launch_max));
    g.rest = (unsigned)std::min<int64_t>(capacity - g.known, walkers);
    return g;
}

// Steps of `rows` rows that a list of `count` rows takes, for every count (near 2^31 rows the sum only fits unsigned).
constexpr int list_steps(int count, int rows) { return (int)(((unsigned)count + (unsigned)rows - 1u) / (unsigned)rows); }

// Step that workgroup `b` of a launch of `grid` workgroups takes of a list of `steps` steps.  Workgroups go to the eight
// dies (XCDs) in turn, each with an L2 of its own, so the steps are dealt out in eight contiguous parts, one per die, each
// in order: neighbouring rows of a list then meet in one L2.  Rows of a link matrix that belong to one host share most of
// their columns: on 10M pages with host locality (d = 128, fp32) the kernel of 16 < k <= 32 reads 16.8 GB per half from
// beyond the L2 instead of 53.6 GB (8.12 -> 7.65 ms; it is bound by its instructions then), 32 < k <= 48 takes
// 3.00 -> 2.83 ms and 8 < k <= 16 3.49 -> 3.39 ms.  Where columns are uniform nothing is lost.  A permutation of
// 0 .. grid - 1 whatever the sizes: the at most seven steps that do not divide, and workgroups beyond the list, keep their place.
constexpr int xcd_step(int b, int grid, int steps) {
    const int chunk = (steps < grid ? steps : grid) >> 3;
    return b < 8 * chunk ? (b & 7) * chunk + (b >> 3) : b;
}

// What workgroup `b` of `grid` (a multiple of eight) takes of a list of `count` rows walked four at a time: the steps blk,
// blk + stride, .. below end.  Each die takes a contiguous eighth of the list, its workgroups in turn.
struct WalkRange { int blk, end, stride; };
constexpr WalkRange walk_range(unsigned b, unsigned grid, int count) {
    const int steps = list_steps(count, 4), part = list_steps(steps, 8), first = (int)(b & 7) * part;
    return {first + (int)(b >> 3), first + part < steps ? first + part : steps, (int)(grid / 8)};
}

// Workgroups (one wavefront each) that walk a list, each in strides of the grid: a multiple of eight, for any list.  Four steps each
// where the list is long: a wavefront loads ahead for its next step, so more steps are better, but with one set of wavefronts
// for the whole list the slowest ones end late, and an empty workgroup costs 0.2 ns.  8 < k <= 16, ms per half, steps per wavefront
// 1 / 3.4 / 7 / 14 / all (fp32, d = 128, 10M pages): 2.99 / 2.70 / 2.72 / 2.75 / 4.02.  hint: steps that an earlier call saw, or -1.
inline unsigned walk_grid(int64_t resident, int64_t capacity, int64_t hint) {
    constexpr int64_t PER_WAVE = 4, LAUNCH_MAX = 0xffffffff / 64 / 8 * 8;
    const int64_t steps = hint < 0 ? capacity : std::min(hint, capacity);
    const int64_t grid = std::max((steps + PER_WAVE - 1) / PER_WAVE, std::min(capacity, resident));
    return (unsigned)std::min((grid + 7) / 8 * 8, LAUNCH_MAX);
}

// The same in whole rounds of as many workgroups as the device holds at a time, so that a short list has no last round of a few workgroups
// with four steps each.  300k rows folded in (d = 128, bf16; 17 024 steps of 16 < k <= 32 on 2048 places): 115 -> 107 us; 40 000 rows of
// 40 entries (d = 64; 10 000 steps of 20 us): the call 225 -> 208 us; one round only, of up to sixteen steps, was slower where a list had more than a few (300k rows of up to 30 entries, d = 128, fp32: 499 -> 579 us).
inline unsigned walk_blocks(int64_t resident, int64_t capacity, int64_t hint) {
    constexpr int64_t PER_WAVE = 4, ROUNDS = 8;
    const int64_t steps = hint < 0 ? capacity : std::min(hint, capacity);
    const int64_t rounds = (steps + PER_WAVE * resident - 1) / (PER_WAVE * resident);
    if (steps > resident && rounds <= ROUNDS) return (unsigned)((rounds * resident + 7) / 8 * 8);
    return walk_grid(resident, capacity, hint);
}

// X = R L^-1 over class lists (transform_lists_kernel), 32 rows per wavefront at a time: workgroups, each of which lays out the matrix
// for itself.  `tiles`: what the lists can hold by their capacities; every one of the `rows` rows is in one of the `lists` lists at most.
// While a workgroup of four wavefronts per compute unit holds all tiles, that is what is launched, otherwise eight share a matrix.
struct TileGrid { unsigned blocks, threads; };
inline TileGrid tile_grid(int num_cu, int64_t tiles, int64_t rows, int lists) {
    tiles = std::min(tiles, rows / 32 + lists);
    const int waves = tiles <= 4 * (int64_t)num_cu ? 4 : 8;
    return {(unsigned)std::min<int64_t>(2 * num_cu, (tiles + waves - 1) / waves), 64u * (unsigned)waves};
}

}  // namespace als
