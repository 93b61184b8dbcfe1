"""Memory of the adjoint's kept states: the budget that all contexts share, what a call gives back, and the same gradients whichever
way the states come."""
import threading

import numpy as np
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, STEPS = 512, 100
SLOT = 15 * 4 * N * N  # one state: 14 populations and phi_prev
MIB = 1 << 20


def cfg():
    c = dict(W.COMMON)
    c.update(nx=N, ny=N, flow=0, inout=0, eps=0.04, seed=(N / 2, N / 2, 20.0), w_init=1.0, U0=0.5)
    return c


def inputs():
    gen = torch.Generator(device="cuda").manual_seed(3)
    U = 0.5 + 0.02 * torch.randn((N, N), generator=gen, device="cuda")
    return U, torch.randn((N, N), generator=gen, device="cuda")


def passes(sim, U, g, stride=0, steps=STEPS):
    sim.init(U)
    S.snowlb_adj_forward(sim.ctx, steps, stride, sim.stream)
    dU = torch.empty_like(g)
    de, du = S.snowlb_adj_backward(sim.ctx, g.data_ptr(), dU.data_ptr(), sim.stream)
    return dU, de, du


def same(a, b):
    return torch.equal(a[0], b[0]) and a[1:] == b[1:]


class Held:
    """Device memory taken since this object was made, in states."""

    def __init__(self):
        torch.cuda.synchronize()
        self.free = torch.cuda.mem_get_info()[0]

    def __call__(self):
        torch.cuda.synchronize()
        return (self.free - torch.cuda.mem_get_info()[0]) / SLOT


def test_budget_of_zero_keeps_checkpoints(monkeypatch):
    """Checkpoints and two segments of ten steps are 30 states, kept states 100 (and the adjoint's own buffers two)."""
    U, g = inputs()
    sims = [S.Sim(cfg()).init(U) for _ in range(2)]
    passes(S.Sim(cfg()), U, g, 10, 20)  # everything that a first pass leaves behind in the process
    monkeypatch.setenv("SNOWLB_ADJ_KEEP_MIB", "0")
    held = Held()
    a = passes(sims[0], U, g)
    assert 29 <= held() <= 40
    monkeypatch.delenv("SNOWLB_ADJ_KEEP_MIB")
    held = Held()
    b = passes(sims[1], U, g)
    assert 99 <= held() <= 110
    assert same(a, b)


def test_kept_states_are_given_back():
    U, g = inputs()
    sim = S.Sim(cfg()).init(U)
    passes(S.Sim(cfg()), U, g, 10, 20)
    held = Held()
    a = passes(sim, U, g)
    assert 99 <= held() <= 110
    b = passes(sim, U, g, 10)
    assert 29 <= held() <= 40
    c = passes(sim, U, g)
    assert 99 <= held() <= 110
    short = passes(sim, U, g, 0, 30)
    assert held() <= 40
    assert same(short, passes(S.Sim(cfg()), U, g, 6, 30))
    assert same(a, b) and same(a, c)
    passes(sim, U, g)
    del sim
    assert held() <= 8


def test_contexts_share_the_budget(monkeypatch):
    """A budget of 150 states: one of two contexts keeps its 100, the other checkpoints, until the first is gone."""
    U, g = inputs()
    sims = [S.Sim(cfg()).init(U) for _ in range(3)]
    passes(S.Sim(cfg()), U, g, 10, 20)
    monkeypatch.setenv("SNOWLB_ADJ_KEEP_MIB", str(150 * SLOT // MIB))
    held = Held()
    a = passes(sims[0], U, g)
    assert 99 <= held() <= 110
    held = Held()
    b = passes(sims[1], U, g)
    b2 = passes(sims[1], U, g)
    assert 29 <= held() <= 40
    del sims[0]
    held = Held()
    c = passes(sims[1], U, g)  # sims[2] of before
    assert 99 <= held() <= 110
    assert same(a, b) and same(a, b2) and same(a, c)


def test_threads_share_the_budget(monkeypatch):
    """Four threads on streams of their own with room for two of them: never more than the budget, and one result."""
    U, g = inputs()
    want = passes(S.Sim(cfg()), U, g, 10)
    sims = [S.Sim(cfg()).init(U) for _ in range(4)]
    monkeypatch.setenv("SNOWLB_ADJ_KEEP_MIB", str(250 * SLOT // MIB))
    held, out, errors = Held(), [None] * 4, []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(3):
                    out[i] = passes(sims[i], U, g)
        except Exception as e:  # reported by the test's own thread
            errors.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    assert held() <= 2 * 100 + 2 * 30 + 4 * 3 + 12
    for o in out:
        assert same(o, want)
    assert np.isfinite(want[1])
