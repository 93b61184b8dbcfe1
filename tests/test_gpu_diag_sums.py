"""The FP64 sums of the diagnostics against sums of the downloaded populations, at numbers of partial sums around the batches in which
the final kernel loads them (32 lanes of 16 partials), and both entry points bitwise the same."""
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("storage,nx,ny", [
    ("fp32", 2, 2), ("fp32", 1024, 31), ("fp32", 1024, 33), ("fp32", 1024, 511), ("fp32", 1024, 512), ("fp32", 1024, 513),
    ("fp32", 1025, 2047), ("fp16", 16, 15), ("fp16", 256, 32), ("bf16", 256, 33), ("fp16", 512, 256), ("bf16", 513, 257),
    ("fp16", 731, 719),
])
@pytest.mark.parametrize("flow", [0, 1])
def test_sums_of_every_lattice_size(storage, nx, ny, flow):
    """A sum passes through at most 36 additions in a lane, 6 and 4 in a workgroup, 64 and 32 in the final kernel: each within
    2^-53 of the sum of magnitudes, so 150 of them; as much again for the reference."""
    c = dict(W.C3)
    c.update(nx=nx, ny=ny, flow=flow, inout=flow, seed=(nx / 2, ny / 2, min(nx, ny) / 4))
    sim = S.Sim(c, storage=storage).init().step(2)
    d = sim.diag()
    g, h, p = (sim.read_populations(k).double() for k in ("g", "h", "phip"))
    want = {"U": g, "phi": h, "phi_prev": p}
    if flow:
        f = sim.read_populations("f").double()
        want.update(rho=f, jx=torch.stack([f[1], -f[3], f[5], -f[6], -f[7], f[8]]),
                    jy=torch.stack([f[2], -f[4], f[5], f[6], -f[7], -f[8]]))
    for k, v in want.items():
        assert abs(d[k] - float(v.sum())) <= 300 * 2.0 ** -53 * float(v.abs().sum()), k
    assert d["n_nonfinite"] == 0
    out = torch.zeros(S.DIAG_COUNT, dtype=torch.float64, device="cuda")
    S.snowlb_diag_noalloc(sim.ctx, out.data_ptr(), sim.stream)
    assert out.tolist() == [d[k] for k in S.DIAG_KEYS]
