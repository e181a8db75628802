"""Steps handed out to the wavefronts of a persistent launch (csrc/step_queue.h), compiled here with the host compiler."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_02194_amd", "csrc")


@pytest.fixture(scope="module")
def queue(tmp_path_factory):
    """times each step is handed out when `waves` wavefronts of `per_block` a workgroup ask in turn until none gets any more"""
    d = tmp_path_factory.mktemp("step_queue")
    src, lib = d / "q.cpp", d / "q.so"
    src.write_text('#include <vector>\n#include "step_queue.h"\n'
                   'extern "C" int run(int steps, int waves, int per_block, int *times) {\n'
                   '    int32_t counters[als::QUEUE_INTS] = {0}; int bad = 0;\n'
                   '    std::vector<als::StepQueue> q;\n'
                   '    for (int w = 0; w < waves; ++w) q.push_back(als::step_queue(counters, steps, w / per_block, waves / per_block, w % per_block, per_block));\n'
                   '    auto look = [](const int32_t *c) { return *c; };\n'
                   '    auto take = [](int32_t *c, int n) { const int v = *c; *c += n; return v; };\n'
                   '    for (bool more = true; more;) { more = false;\n'
                   '        for (auto &w : q) { const int s = w.next(look, take); if (s < 0) { bad += w.next(look, take) >= 0; continue; }\n'
                   '            more = true; if (s >= steps) ++bad; else ++times[s]; } }\n'
                   '    return bad; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", str(lib), str(src)])
    f = ctypes.CDLL(str(lib)).run

    def call(steps, waves, per_block):
        times = (ctypes.c_int * max(steps, 1))()
        return f(steps, waves, per_block, times), list(times)[:steps]
    return call


@pytest.mark.parametrize("waves,per_block", [(8, 1), (64, 8), (192, 8), (2048, 8)])
@pytest.mark.parametrize("steps", [0, 1, 7, 8, 9, 63, 64, 65, 511, 513, 2047, 131_077])
def test_every_step_is_handed_out_once(queue, steps, waves, per_block):
    bad, times = queue(steps, waves, per_block)
    assert bad == 0 and all(t == 1 for t in times)
