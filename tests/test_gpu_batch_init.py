"""The initial state of a batch, written by one launch over all its tiles, against each lattice's own."""
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("flow", [0, 1])
@pytest.mark.parametrize("sizes", [[(64, 4), (65, 5)], [(2, 2), (130, 9), (1, 70)], [(63, 3)]])
def test_batch_initial_state_is_bitwise_each_lattices_own(storage, flow, sizes):
    """Sizes at and one past a 64 x 4 tile, the smallest ones, and a batch of one; each lattice with a seed, U0 and
    width of its own; again after steps have moved the batch to its other copy."""
    cfgs = []
    for i, (nx, ny) in enumerate(sizes):
        c = dict(W.C3)
        c.update(nx=max(nx, 2), ny=max(ny, 2), flow=flow, inout=flow, seed=(nx / 3, ny / 2, 2.0 + i), U0=0.4 + 0.05 * i,
                 w_init=1.0 + 0.5 * i)
        cfgs.append(c)
    b = S.Batch(cfgs, storage)
    for steps in (0, 3):
        b.init().step(steps)
        if steps:
            b.init()
        for i, c in enumerate(cfgs):
            one = S.Sim(c, storage=storage).init()
            for f in ("phi", "U") + (("rho", "ux") if flow else ()):
                assert torch.equal(b.read(i, f), one.read(f)), (i, f)
    b.step(2)
    for i, c in enumerate(cfgs):
        assert torch.equal(b.read(i, "phi"), S.Sim(c, storage=storage).init().step(2).read("phi"))
