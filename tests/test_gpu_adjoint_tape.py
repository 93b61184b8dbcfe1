"""The adjoint with every state kept (checkpoint stride left to the library) against checkpointed runs, bitwise, and
the reverse tiles' rows on a lattice that is ragged against them."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cfg_of(nx, ny, R=6.0):
    c = dict(W.COMMON)
    c.update(nx=nx, ny=ny, flow=0, inout=0, eps=0.04, seed=(nx / 2, ny / 2, R), w_init=1.0, U0=0.5)
    return c


def backward(sim, gphi):
    dU = torch.empty_like(gphi)
    de, du = S.snowlb_adj_backward(sim.ctx, gphi.data_ptr(), dU.data_ptr(), sim.stream)
    return dU.cpu().numpy(), de, du


@pytest.mark.parametrize("n,tile", [(1, 0), (2, 0), (10, 0), (41, 3), (100, 0)])
def test_kept_states_match_checkpoints(n, tile):
    """Kept states (stride 0) against checkpoints every ceil(sqrt n) and every 3 steps: phi_T, the step count and
    every gradient are the same bits; again after a second forward pass with fewer steps on the same context, and
    after a change of eps between the passes (both recompute the intervals with the new eps)."""
    cfg = cfg_of(70, 37)
    rng = np.random.default_rng(n)
    U = torch.from_numpy((0.5 + 0.02 * rng.standard_normal((37, 70))).astype(np.float32)).cuda()
    gphi = torch.from_numpy(rng.standard_normal((37, 70)).astype(np.float32)).cuda()
    st = int(np.ceil(np.sqrt(n)))
    out = []
    for stride in (0, st, 3):
        sim = S.Sim(cfg)
        sim.set_tile(tile)
        got = []
        for steps in (n, max(1, n - 1)):
            sim.init(U)
            S.snowlb_adj_forward(sim.ctx, steps, stride, sim.stream)
            got += [sim.read("phi").cpu().numpy(), sim.step_count, *backward(sim, gphi)]
        sim.init(U)
        S.snowlb_adj_forward(sim.ctx, n, stride, sim.stream)
        sim.step(3)  # the context moves on; the kept states do not
        got += [*backward(sim, gphi)]
        if stride != 3:  # with another stride the intervals recomputed after a change of eps are others
            S.snowlb_set_eps(sim.ctx, 0.06)
            got += [*backward(sim, gphi)]
        out.append(got)
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)


def test_tall_reverse_tiles_on_a_ragged_lattice():
    """65 x 1801 cells: 226 tiles of 64 x 16, enough of the 256 that fill the chip to be chosen, the last column
    one cell wide and the last row nine high.  Every gradient against the oracle's discrete adjoint (1e-3, as
    for the other ragged lattices)."""
    nx, ny, steps = 65, 1801, 12
    cfg = cfg_of(nx, ny)
    rng = np.random.default_rng(5)
    U = (0.5 + 0.02 * rng.standard_normal((ny, nx))).astype(np.float32).astype(np.float64)
    p = oracle.Params.from_dict(cfg)
    target = oracle.final_phi(dataclasses.replace(p, eps=0.06), cfg["seed"], 1.0, 0.55 + 0 * U, steps)
    _, dUo, deo, _ = oracle.adjoint(p, cfg["seed"], 1.0, U, target, steps)
    sim = S.Sim(cfg).init(torch.from_numpy(U).float())
    S.snowlb_adj_forward(sim.ctx, steps, 0, sim.stream)
    seed = (2 * (sim.read("phi").double() - torch.from_numpy(target).cuda())).float().contiguous()
    dU, de, _ = backward(sim, seed)
    scale = float(np.abs(dUo).max())
    print("  65 x 1801: deps %.6e / %.6e, dU max err %.3e of %.3e" % (de, deo, np.abs(dU - dUo).max(), scale))
    assert abs(de - deo) <= 1e-3 * abs(deo)
    assert np.abs(dU - dUo).max() <= 1e-3 * scale
