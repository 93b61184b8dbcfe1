"""The default tile of the 2D step: two blocks wide or high for 16-bit lattices larger than the last-level
cache, else one."""
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cfg_of(nx, ny, flow):
    c = dict(W.C3)
    c.update(nx=nx, ny=ny, seed=(nx / 2, ny / 2, min(nx, ny) / 4), flow=flow, inout=flow)
    return c


@pytest.mark.parametrize("nx,ny,flow,storage,name", [
    (1344, 2001, 1, "fp16", "128x4"),   # 21 blocks: one lane in 22 idle
    (1279, 2001, 1, "bf16", "128x4"),   # 20
    (1216, 2001, 1, "fp16", "64x8"),    # 19: one in 20
    (2113, 2250, 0, "bf16", "128x4"),   # 34 blocks, the last one cell wide
    (65, 20003, 1, "fp16", "128x4"),    # 2 blocks, the last one cell wide
    (64, 38001, 1, "fp16", "64x8"),     # one block
    (190, 15001, 0, "bf16", "64x4"),    # 3 blocks, in the cache
    (1000, 1000, 1, "fp16", "64x4"),
    (1088, 2301, 1, "fp32", "64x4"),
])
def test_default_tile_and_its_results(nx, ny, flow, storage, name):
    """The rule at its edges, and every field after five steps bitwise equal to the 64 x 4 tile's."""
    sim = S.Sim(cfg_of(nx, ny, flow), storage=storage).init().step(5)
    assert S.snowlb_tile_name(sim.tile) == name
    one = S.Sim(cfg_of(nx, ny, flow), storage=storage)
    one.set_tile(0)
    assert one.tile == 0
    one.init().step(5)
    for f in ("phi", "U") + (("rho", "ux", "uy") if flow else ()):
        assert torch.equal(sim.read(f), one.read(f)), f


def test_default_tile_of_a_batch():
    """A batch decides on all its lattices together; its members equal solo runs of 64 x 4 tiles bitwise."""
    cfgs = [cfg_of(800 + 37 * i, 700 + 29 * i, 1) for i in range(4)]
    b = S.Batch(cfgs, "fp16").init().step(5)
    assert S.snowlb_tile_name(b.tile) == "128x4"
    for i, c in enumerate(cfgs):
        one = S.Sim(c, storage="fp16").init()
        assert one.tile == 0  # each by itself fits in the cache
        one.step(5)
        assert torch.equal(b.read(i, "phi"), one.read("phi"))
    assert S.snowlb_tile_name(S.Batch([cfg_of(150 + 7 * i, 1150, 1) for i in range(12)], "fp16").tile) == "64x8"
