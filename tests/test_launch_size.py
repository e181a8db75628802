"""The launch sizes of the row lists (host arithmetic of csrc/launch_size.h), compiled here with the host compiler."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_02194_amd", "csrc")


@pytest.fixture(scope="module")
def step_grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_size")
    src, lib = d / "l.cpp", d / "l.so"
    src.write_text('#include "launch_size.h"\n'
                   'extern "C" void grid(int cu, int threads, int64_t cap, int64_t hint, int per_cu, int64_t blind, unsigned *out) {\n'
                   '    const als::StepGrid g = als::step_grid(cu, threads, cap, hint, per_cu, blind); out[0] = g.known; out[1] = g.rest; }\n'
                   'extern "C" void beside(int cu, int threads, int64_t cap, int64_t hint, int per_cu, int64_t blind, int64_t other, unsigned *out) {\n'
                   '    const als::StepGrid g = als::step_grid(cu, threads, cap, hint, per_cu, blind, other); out[0] = g.known; out[1] = g.rest; }\n'
                   'extern "C" unsigned walk(int64_t resident, int64_t cap, int64_t hint) { return als::walk_grid(resident, cap, hint); }\n'
                   'extern "C" unsigned walk_blocks(int64_t resident, int64_t cap, int64_t hint) { return als::walk_blocks(resident, cap, hint); }\n'
                   'extern "C" void tiles(int cu, int64_t tiles, int64_t rows, int lists, unsigned *out) {\n'
                   '    const als::TileGrid g = als::tile_grid(cu, tiles, rows, lists); out[0] = g.blocks; out[1] = g.threads; }\n'
                   'extern "C" int xcd(int b, int grid, int steps) { return als::xcd_step(b, grid, steps); }\n'
                   'extern "C" int list_steps(int count, int rows) { return als::list_steps(count, rows); }\n'
                   'extern "C" void walk_range(int b, int grid, int count, int *out) {\n'
                   '    const als::WalkRange w = als::walk_range(b, grid, count); out[0] = w.blk; out[1] = w.end; out[2] = w.stride; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", str(lib), str(src)])
    beside.f = ctypes.CDLL(str(lib)).beside
    beside.f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    tile_grid.f = ctypes.CDLL(str(lib)).tiles
    tile_grid.f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_void_p]
    walk_grid.f = ctypes.CDLL(str(lib)).walk
    walk_grid.f.argtypes, walk_grid.f.restype = [ctypes.c_int64] * 3, ctypes.c_uint
    walk_blocks.f = ctypes.CDLL(str(lib)).walk_blocks
    walk_blocks.f.argtypes, walk_blocks.f.restype = [ctypes.c_int64] * 3, ctypes.c_uint
    xcd.f = ctypes.CDLL(str(lib)).xcd
    list_steps.f = ctypes.CDLL(str(lib)).list_steps
    walk_range.f = ctypes.CDLL(str(lib)).walk_range
    f = ctypes.CDLL(str(lib)).grid
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_void_p]

    def call(threads, cap, hint, per_cu=32, blind=1 << 22, cu=256):
        out = (ctypes.c_uint * 2)()
        f(cu, threads, cap, hint, per_cu, blind, out)
        return int(out[0]), int(out[1])
    return call


def beside(threads, cap, hint, other, per_cu=8, blind=1 << 20, cu=256):
    out = (ctypes.c_uint * 2)()
    beside.f(cu, threads, cap, hint, per_cu, blind, other, out)
    return int(out[0]), int(out[1])


def tile_grid(tiles, rows, lists, cu=256):
    out = (ctypes.c_uint * 2)()
    tile_grid.f(cu, tiles, rows, lists, out)
    return int(out[0]), int(out[1])


def xcd(b, grid, steps):
    return xcd.f(b, grid, steps)


def list_steps(count, rows):
    return list_steps.f(count, rows)


def walk_range(b, grid, count):
    out = (ctypes.c_int * 3)()
    walk_range.f(b, grid, count, out)
    return tuple(out)


def walk_grid(resident, cap, hint):
    return walk_grid.f(resident, cap, hint)


def walk_blocks(resident, cap, hint):
    return walk_blocks.f(resident, cap, hint)


SIZES = [0, 1, 4095, 4096, 4097, 100_000, (1 << 24) - 1, 1 << 24, 25_000_000, 50_000_000, (1 << 26) - 1, 1 << 26, (1 << 31) - 1]


@pytest.mark.parametrize("threads", [64, 128, 256])
def test_the_two_forms_cover_the_list_and_fit_one_launch(step_grid, threads):
    for cap in SIZES:
        for hint in [-1] + SIZES:
            known, rest = step_grid(threads, cap, hint)
            assert known <= cap and (known + rest) * threads < 1 << 32
            assert known + rest == cap or rest == 256 * 32  # what the first form leaves is walked by the second
            if cap <= 4096:
                assert (known, rest) == (cap, 0)
            elif hint >= 0 and (hint + 256 * 32) * threads < 1 << 32:
                assert known == min(hint, cap)  # a hint is followed as far as a launch can hold it
            elif hint < 0:
                assert known == min(cap, 1 << 22)


@pytest.mark.parametrize("threads", [64, 128, 256])
@pytest.mark.parametrize("segments", [0, 1, 4096, 4097, 10_000, 1 << 15])
def test_two_lists_that_share_a_launch_fit_it_together(step_grid, threads, segments):
    """Rows solved whole and segments of long rows, as many as a call before saw: a launch for the first parts."""
    other, _ = step_grid(threads, 1 << 15, segments, per_cu=8, blind=1 << 15)
    for cap in SIZES:
        for hint in [-1] + SIZES:
            known, rest = beside(threads, cap, hint, other)
            assert (known + other) * threads < 1 << 32
            assert known <= cap and (known + rest == cap or rest == 256 * 8)
            alone, _ = step_grid(threads, cap, hint, per_cu=8, blind=1 << 20)
            assert known == alone or known + rest + other == 0xffffffff // threads  # no fewer than a launch can hold


def test_a_long_list_of_small_workgroups_is_launched_whole(step_grid):
    """2.2e7 steps of four rows (a 100M-row epoch): more than 2^24 workgroups of 64 threads are one launch."""
    assert step_grid(64, 25_000_000, 22_000_000) == (22_000_000, 8192)


def test_a_long_list_of_large_workgroups_stays_below_the_launch_limit(step_grid):
    known, rest = step_grid(256, 50_000_000, 50_000_000)
    assert known < 1 << 24 and rest == 8192


@pytest.mark.parametrize("grid", [1, 7, 8, 9, 63, 64, 1000, 4097])
def test_steps_are_dealt_out_once_each_in_eight_parts(step_grid, grid):
    for steps in [0, 1, 7, 8, grid - 1, grid, grid + 1, 10 * grid]:
        order = [xcd(b, grid, steps) for b in range(grid)]
        assert sorted(order) == list(range(grid))
        for die in range(8):  # what one die gets of the divisible part is contiguous and in order
            part = [s for s in order[die::8] if s < min(steps, grid) // 8 * 8]
            assert part == list(range(part[0], part[0] + len(part))) if part else True


def test_a_walked_list_gets_enough_workgroups_and_no_more_than_a_launch_holds(step_grid):
    for cap in SIZES[1:]:
        for hint in [-1] + SIZES:
            g = walk_grid(3072, cap, hint)
            assert g % 8 == 0 and g > 0 and g * 64 < 1 << 32
            steps = cap if hint < 0 else min(cap, hint)
            assert g >= min(cap, 3072) and (g >= steps / 4 or g * 64 >= (1 << 32) - 512)  # at most four steps each, if a launch can hold that
            assert g <= max(steps / 4, min(cap, 3072)) + 8


@pytest.mark.parametrize("resident", [8, 1000, 2048, 3072])
def test_a_short_walked_list_gets_whole_rounds_of_what_the_device_holds(step_grid, resident):
    for cap in SIZES[1:] + [resident, resident + 1, 4 * resident, 4 * resident + 1, 32 * resident, 32 * resident + 1]:
        for hint in [-1] + SIZES:
            g, steps = walk_blocks(resident, cap, hint), cap if hint < 0 else min(cap, hint)
            assert g % 8 == 0 and 0 < g and g * 64 < 1 << 32
            if steps <= resident or steps > 32 * resident:
                assert g == walk_grid(resident, cap, hint)
            else:  # one to eight rounds of at most four steps a wavefront, and not a round more than that takes
                rounds = -(-steps // (4 * resident))
                assert rounds * resident <= g < rounds * resident + 8 and steps <= 4 * g and 1 <= rounds <= 8


@pytest.mark.parametrize("rows", [1, 4, 8, 16])
def test_steps_of_a_list_up_to_the_longest_range(step_grid, rows):
    """count + rows - 1 would be negative for the longest lists, which a kernel then takes for empty ones."""
    for count in [0, 1, rows - 1, rows, rows + 1, 1000, (1 << 31) - 1 - rows, (1 << 31) - rows, (1 << 31) - 2, (1 << 31) - 1]:
        assert list_steps(count, rows) == -(-count // rows)


@pytest.mark.parametrize("count", [0, 1, 4, 5, 31, 32, 33, 100_003, (1 << 31) - 4, (1 << 31) - 3, (1 << 31) - 1])
def test_a_walk_covers_its_list_once(step_grid, count):
    """The parts of the eight dies join without a gap, and the workgroups of a die take every place of a stride."""
    steps = -(-count // 4)
    for grid in [8, 64, 1 << 20, walk_grid(3072, steps, -1) or 8]:
        end = 0
        for die in range(8):
            first, stop, stride = walk_range(die, grid, count)
            assert first == min(end, steps) or first >= stop
            end = max(end, stop)
            assert stride == grid // 8
            for w in {0, 1, stride - 1} & set(range(stride)):
                assert walk_range(die + 8 * w, grid, count) == (first + w, stop, stride)
        assert end == steps


@pytest.mark.parametrize("rows", [1, 31, 33, 256, 9000, 15_000, 32_000, 33_000, 300_000, 50_000_000, (1 << 31) - 1])
@pytest.mark.parametrize("mean", [1, 12, 40])
def test_the_pass_over_the_lists_gets_no_more_workgroups_than_rows_need(step_grid, rows, mean):
    """Every list can hold all rows, or as many as the entries allow, but a row is in one of them only."""
    caps = [min(rows, rows * mean // least + 1) for least in (1, 5, 9, 17, 33, 49, 65, 81, 97, 113)]
    blocks, threads = tile_grid(sum(-(-c // 32) for c in caps), rows, len(caps))
    waves = threads // 64
    assert waves in (4, 8) and 1 <= blocks <= 512
    assert blocks * waves < rows / 32 + len(caps) + waves  # one tile per list that is not full
    assert blocks == 512 or blocks * waves >= -(-rows // 32)  # a tile a wavefront, or all that find a place at a time
    assert waves == 8 or blocks <= 256
