"""The places of rows that a wavefront copies to LDS (csrc/row_copy.h), compiled here with the host compiler."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_02194_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_copy")
    src, out = d / "r.cpp", d / "r.so"
    src.write_text('#include "row_copy.h"\n'
                   'extern "C" int columns(int d) { return als::columns_per_lane(d); }\n'
                   'extern "C" int holds(int d, int lane) { return als::holds_columns(d, lane); }\n'
                   'extern "C" int stride(int d) { return als::row_copy_stride(d); }\n'
                   'extern "C" int place(int d, int n, int lane) { return als::row_copy_place(d, n, lane); }\n')
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", str(out), str(src)])
    return ctypes.CDLL(str(out))


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("rows", [8, 16])
def test_every_place_of_a_copied_row_is_written_by_one_lane(lib, d, rows):
    """Stores of different lanes have no order: no two may go to one place, and none beyond its row."""
    cpl = lib.columns(d)
    written = {}
    for n in range(rows):
        for lane in range(64):
            if lib.holds(d, lane):
                for c in range(cpl):
                    at = lib.place(d, n, lane) + c
                    assert n * lib.stride(d) <= at < n * lib.stride(d) + d
                    assert written.setdefault(at, (n, lane)) == (n, lane)
    assert len(written) == rows * d
