"""Graph replay of the steps, bitwise against direct launches: from either copy, with remainders, and across a change of tile or
launch mode, in two and three dimensions and for batches.  The graphs are short here, so that every call replays several."""
import os

import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cfg2(nx, ny, **kw):
    c = dict(W.C3)
    c.update(nx=nx, ny=ny, seed=(nx / 3, ny / 2, min(nx, ny) / 5))
    c.update(kw)
    return c


def pops(sim):
    return [sim.read_populations(k) for k in ("f", "g", "h", "phip")]


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def run(monkeypatch, sim, calls, steps):
    """The calls with graphs of `steps` steps (0: direct launches); the state after each of them."""
    monkeypatch.setenv("SNOWLB_GRAPH_STEPS", str(steps or 2))
    monkeypatch.setenv("SNOWLB_NO_GRAPH", "0" if steps else "1")
    out = []
    for n in calls:
        if isinstance(n, tuple):
            sim.set_tile(n[0])
            sim.set_grid_mode(n[1])
        else:
            sim.step(n)
            out.append((sim.step_count, pops(sim)))
    return out


# from copy 0: 8 (and 32); from copy 1 after an odd call: 9 = 1 + 8, 33; odd remainders: 10 + 1; other tiles and modes between
CALLS = [8, 11, 9, 32, 1, 33, 20, (3, 0), 16, (1, 2), 21, 8, (0, 1), 12]


@pytest.mark.parametrize("steps", [2, 4, 8])
@pytest.mark.parametrize("storage", ["fp32", "bf16"])
def test_replay_matches_direct_launches_2d(storage, steps, monkeypatch):
    cfg = cfg2(100, 90)
    want = run(monkeypatch, S.Sim(cfg, storage=storage).init(), CALLS, 0)
    got = run(monkeypatch, S.Sim(cfg, storage=storage).init(), CALLS, steps)
    for (n, a), (m, b) in zip(want, got):
        assert n == m and same(a, b), n


@pytest.mark.parametrize("steps", [2, 8])
def test_replay_matches_direct_launches_3d(steps, monkeypatch):
    cfg = dict(W.F4_3D)
    cfg.update(nx=70, ny=20, nz=12, seed=(20.0, 10.0, 6.0, 4.0))
    calls = [n for n in CALLS if not isinstance(n, tuple)]
    want = run(monkeypatch, S.Sim3D(cfg).init(), calls, 0)
    got = run(monkeypatch, S.Sim3D(cfg).init(), calls, steps)
    for (n, a), (m, b) in zip(want, got):
        assert n == m and same(a, b), n


@pytest.mark.parametrize("steps", [2, 8])
def test_replay_matches_direct_launches_batch(steps, monkeypatch):
    cfgs = [cfg2(100 + 13 * i, 60 + 7 * i) for i in range(4)]

    def go(k):
        monkeypatch.setenv("SNOWLB_GRAPH_STEPS", str(k or 2))
        monkeypatch.setenv("SNOWLB_NO_GRAPH", "0" if k else "1")
        b = S.Batch(cfgs).init()
        for n in CALLS:
            if isinstance(n, tuple):
                b.set_tile(*n)
            else:
                b.step(n)
        return b.step_count, [b.read(i, f) for i in range(4) for f in ("phi", "U", "rho", "ux", "uy")]

    n, want = go(0)
    m, got = go(steps)
    assert n == m and same(want, got)


def test_replays_on_streams_of_their_own(monkeypatch):
    """Contexts on several streams, with the default graphs: each as the same context alone with direct launches."""
    cfgs = [cfg2(90 + 20 * i, 80 + 10 * i) for i in range(4)]
    monkeypatch.setenv("SNOWLB_NO_GRAPH", "1")
    want = [pops(S.Sim(c).init().step(64).step(97).step(40)) for c in cfgs]
    monkeypatch.setenv("SNOWLB_NO_GRAPH", "0")
    sims, streams = [S.Sim(c) for c in cfgs], [torch.cuda.Stream() for _ in cfgs]
    for n in (0, 64, 97, 40):
        for sim, st in zip(sims, streams):
            with torch.cuda.stream(st):
                sim.step(n) if n else sim.init()
    torch.cuda.synchronize()
    assert os.environ["SNOWLB_NO_GRAPH"] == "0"
    for sim, w in zip(sims, want):
        assert same(pops(sim), w)


@pytest.mark.parametrize("n", [20, 64, 256])
def test_steps_inside_a_callers_capture(n):
    """A caller's capture of a call long enough for the library's own graphs records single steps: three replays, with eager work
    between them, equal as many eager calls."""
    cfg, cfg3 = cfg2(100, 90), dict(W.F4_3D)
    cfg3.update(nx=70, ny=20, nz=12, seed=(20.0, 10.0, 6.0, 4.0))
    for make in (lambda: S.Sim(cfg), lambda: S.Sim3D(cfg3)):
        want = make().init().step(2)
        sim = make().init().step(2)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            sim.step(n)
        for _ in range(3):
            graph.replay()
            want.step(n)
            assert same(pops(sim), pops(want))
            sim.step(2)
            want.step(2)
            torch.cuda.synchronize()
        assert same(pops(sim), pops(want))
