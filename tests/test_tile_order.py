"""The tile order a single lattice's step computes (StepGeom::tile_at) and the block order of the 3D step (block_of)
against the plain loops that define them, on the host: row order and strips of every width, the last strip
narrower or not; slabs of equal and of unequal height."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "snowlb_internal.h"
#include "snowlb3d_internal.h"
using namespace snowlb;
static int check(int ntx, int nty, int W) {
    StepGeom g;
    g.set_lattice(ntx, nty, W);
    if (g.ntiles != ntx * nty) return 1;
    int t = 0;
    for (int s0 = 0; s0 < ntx; s0 += W)
        for (int j = 0; j < nty; ++j)
            for (int i = s0; i < ntx && i < s0 + W; ++i, ++t) {
                int ti, tj;
                g.tile_at(t, ti, tj);
                if (ti != i || tj != j) {
                    std::printf("ntx %d nty %d strip %d tile %d: (%d, %d) instead of (%d, %d)\n", ntx, nty, W, t, ti, tj, i, j);
                    return 1;
                }
            }
    return t == g.ntiles ? 0 : 1;
}
static int check3(int nbx, int nby, int nbz) {
    snowlb3d::Dom3 d{};
    d.nbx = nbx;
    d.nby = nby;
    d.nbz = nbz;
    snowlb3d::set_block_order(d);
    const int slabs = nby >= 8 ? 8 : 1;
    int t = 0;
    for (int s = 0; s < slabs; ++s)
        for (int k = 0; k < nbz; ++k)
            for (int j = (int)((int64_t)s * nby / slabs); j < (int)((int64_t)(s + 1) * nby / slabs); ++j)
                for (int i = 0; i < nbx; ++i, ++t) {
                    int bx, by, bz;
                    snowlb3d::block_of(d, t, bx, by, bz);
                    if (bx != i || by != j || bz != k) {
                        std::printf("%d x %d x %d block %d\n", nbx, nby, nbz, t);
                        return 1;
                    }
                }
    return t == nbx * nby * nbz ? 0 : 1;
}
int main() {
    int bad = 0;
    for (int nbx : {1, 2, 3, 4, 8})
        for (int nby : {1, 2, 7, 8, 9, 15, 16, 17, 51, 64, 67})
            for (int nbz : {1, 2, 5, 64}) bad += check3(nbx, nby, nbz);
    bad += check3(1, 32768, 1) + check3(1024, 9, 3) + check3(1, 8, 16384);
    for (int ntx = 1; ntx <= 20; ++ntx)
        for (int nty : {1, 2, 3, 7, 64, 65})
            for (int W = 1; W <= ntx; ++W) bad += check(ntx, nty, W);
    for (int W : {1, 8, 16, 255, 1023, 1024}) bad += check(1024, 300, W);  // 65536 cells in x
    bad += check(1, 32768, 1) + check(109, 1673, 109) + check(109, 1673, 28) + check(109, 1673, 8);
    std::mt19937 r(1);
    for (int k = 0; k < 2000000; ++k) {  // the division itself over its whole range
        const uint32_t n = r() >> (1 + r() % 31), d = 1 + (r() >> (1 + r() % 31));
        const FastDiv f = fast_div(d);
        bad += div_by(n, f.m, f.code) != n / d;
    }
    for (uint32_t d : {1u, 2u, 3u, 5u, 641u, 65535u, 65536u, 0x7fffffffu})
        for (uint32_t n : {0u, 1u, d - 1, d, 0x7ffffffeu, 0x7fffffffu}) {
            const FastDiv f = fast_div(d);
            bad += div_by(n, f.m, f.code) != n / d;
        }
    return bad ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_computed_tile_order_matches_the_loops(tmp_path):
    src = tmp_path / "tiles.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "tiles"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_2101_07163_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
