"""The batches of a top-k call (host arithmetic of csrc/topk_batch.h), compiled here with the host compiler."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_02194_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("topk_batch")
    src, out = d / "b.cpp", d / "b.so"
    src.write_text('#include "topk_batch.h"\n'
                   'extern "C" int64_t batch(int64_t q, int64_t per, int64_t group, int64_t limit) { return als::topk_batch(q, per, group, limit); }\n'
                   'extern "C" int64_t smaller(int64_t b) { return als::topk_smaller_batch(b); }\n')
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", str(out), str(src)])
    lib = ctypes.CDLL(str(out))
    for f in (lib.batch, lib.smaller):
        f.restype = ctypes.c_int64
    lib.batch.argtypes = [ctypes.c_int64] * 4
    lib.smaller.argtypes = [ctypes.c_int64]
    return lib


LIMIT = 3 << 29


@pytest.mark.parametrize("group", [384, 512])
def test_batches_fit_the_launch_and_the_workspace(lib, group):
    for queries in (1, 63, 64, group, group + 1, 4096, 100_003, (1 << 24) - 1, 1 << 24, 20_000_000, 1 << 31):
        for per in (0, 64, 4096, 312_576, 1 << 20, LIMIT, 4 * LIMIT):
            b = lib.batch(queries, per, group, LIMIT)
            assert 1 <= b <= queries and (b == queries or b % group == 0)
            assert b * 256 < 1 << 32  # one workgroup of 256 threads per query
            assert b * per <= LIMIT or b <= group


def test_smaller_batches_end(lib):
    for b in (1, 63, 64, 65, 127, 128, 384, 4096, 4097, 16_776_960):
        steps = 0
        while lib.smaller(b) != b:
            n = lib.smaller(b)
            assert 64 <= n < b
            b, steps = n, steps + 1
        assert b <= 64 and steps <= 20
