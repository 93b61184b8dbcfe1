"""The bits of 16-bit populations as a write stores them, against the same arithmetic in numpy."""
import numpy as np
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NX, NY = 257, 131
W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=np.float32).reshape(9, 1, 1)
I9 = np.array([2.25] + [9.0] * 4 + [36.0] * 4, dtype=np.float64).reshape(9, 1, 1)
W5 = np.array([1 / 3] + [1 / 6] * 4, dtype=np.float32).reshape(5, 1, 1)
I5 = np.array([3.0] + [6.0] * 4, dtype=np.float64).reshape(5, 1, 1)


def read_back(d16, w, ref):
    """fma(w, d, w ref) in FP32 (the products are exact in FP64)."""
    wr = (w * ref).astype(np.float32).astype(np.float64)
    return (w.astype(np.float64) * d16.astype(np.float64) + wr).astype(np.float32)


@pytest.mark.parametrize("flow", [0, 1])
def test_written_fp16_states(flow):
    """The deviation p / w - m of f and g (m = 0 after a write) is rounded to FP32 and then to 16 bits, that of h (m = phi_prev) once,
    from the fused multiply-add.  33667 cells of 23 populations, of which a few in a thousand tell the two apart."""
    rng = np.random.default_rng(4)
    c = dict(W.C3)
    c.update(nx=NX, ny=NY, flow=flow, inout=0, u_in=0.0, seed=(NX / 2, NY / 2, 20.0))
    sim = S.Sim(c, storage="fp16").init()
    phip = rng.standard_normal((NY, NX)).astype(np.float32)
    sim.write_populations("phip", torch.from_numpy(phip))
    told = 0
    for name, w, iw, ref in (("f", W9, I9, 0.0), ("g", W5, I5, 0.0), ("h", W9, I9, phip)):
        if name == "f" and not flow:
            continue
        p = (w * (1.0 + 0.5 * rng.standard_normal((len(w), NY, NX)))).astype(np.float32)
        sim.write_populations(name, torch.from_numpy(p))
        got = sim.read_populations(name).cpu().numpy()
        ref = np.float32(ref)
        e = p.astype(np.float64) * iw - ref.astype(np.float64)
        once, twice = e.astype(np.float16), e.astype(np.float32).astype(np.float16)
        told += int((once != twice).sum())
        want = read_back(once if name == "h" else twice, w, ref)
        assert np.array_equal(got, want), (name, int((got != want).sum()))
    assert told > 10
