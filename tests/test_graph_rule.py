"""Which calls of the step replay captured graphs: whole graphs have to cover four fifths of the call, and eight of them of a call
on a large lattice."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "snowlb_graph.h"
using snowlb::replays_graphs;
int main() {
    struct { int n, K, par, want; } t[] = {
        {0, 32, 0, 0}, {1, 32, 0, 0}, {31, 32, 0, 0}, {32, 32, 0, 1}, {40, 32, 0, 1}, {41, 32, 0, 0}, {50, 32, 0, 0},
        {63, 32, 0, 0}, {64, 32, 0, 1}, {80, 32, 0, 1}, {81, 32, 0, 0}, {96, 32, 0, 1}, {100, 32, 0, 1}, {121, 32, 0, 0},
        {128, 32, 0, 1}, {255, 32, 0, 1}, {256, 32, 0, 1}, {32, 32, 1, 0}, {33, 32, 1, 1}, {0, 32, 1, 0}, {64, 32, 1, 0},
        {65, 32, 1, 1}, {2, 2, 0, 1}, {3, 2, 1, 0}, {5, 2, 1, 1}, {0x7fffffff, 32, 1, 1}, {0x7fffffff, 0x7ffffffe, 0, 1},
    };
    int bad = 0;
    for (const auto& r : t)
        for (int64_t cells : {int64_t(4), int64_t(1) << 17, (int64_t(1) << 17) + 1, int64_t(1) << 27}) {
            const bool want = r.want && (cells <= 131072 || (r.n - r.par) / r.K >= 8);
            if (replays_graphs(r.n, r.K, r.par, cells) != want) {
                std::printf("%d steps, graphs of %d, copy %d, %lld cells\n", r.n, r.K, r.par, (long long)cells);
                ++bad;
            }
        }
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_which_calls_replay_graphs(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem",
                           "/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2101_07163_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
