"""Persistent grids (launch modes 1, 3 and 5) with more tiles than resident workgroups: every result is bitwise that of one
workgroup per tile."""
import ctypes

import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def step_grid(tile, ntiles, storage, flow, inout, reach):
    fn = getattr(S.lib(), "_ZN6snowlb9step_gridEiiiiii")  # snowlb::step_grid
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_int] * 6
    return fn(tile, ntiles, storage, flow, inout, reach)


def tile_shape(tile):
    return tuple(int(v) for v in S.snowlb_tile_name(tile).split("x"))


def cfg_of(nx, ny, flow, inout, stencil):
    c = dict(W.C3)
    c.update(nx=nx, ny=ny, flow=flow, inout=inout, stencil=stencil, seed=(nx / 2, ny / 2, min(nx, ny) / 4))
    if not inout:
        c.update(u_in=0.0)
    return c


@pytest.mark.parametrize("nx,ny,flow,inout,stencil,storage", [
    (1100, 901, 1, 1, 4, "fp32"),    # in the last-level cache
    (1601, 1203, 1, 1, 4, "fp32"),   # from HBM with flow
    (1701, 1403, 0, 0, 4, "fp32"),   # from HBM without
    (1100, 901, 0, 0, 8, "fp32"),
    (1601, 1203, 1, 0, 8, "fp32"),
    (1100, 901, 1, 1, 4, "fp16"),
    (1667, 1503, 1, 0, 8, "bf16"),   # from HBM
])
def test_persistent_grids_are_bitwise_the_same(nx, ny, flow, inout, stencil, storage):
    cfg = cfg_of(nx, ny, flow, inout, stencil)
    gen = torch.Generator(device="cuda").manual_seed(nx)
    U = 0.5 + 0.02 * torch.randn((ny, nx), generator=gen, device="cuda")
    names = (("f",) if flow else ()) + ("g", "h", "phip")
    ref = None
    for tile in range(S.snowlb_tile_count()):
        tx, ty = tile_shape(tile)
        tiles = -(-nx // tx) * -(-ny // ty)
        grid = step_grid(tile, tiles, S.STORAGES[storage], flow, inout, 2 if stencil == 8 else 1)
        assert grid < tiles and tiles % grid, (tile, tiles, grid)
        for mode in (0, 1, 3, 5):
            sim = S.Sim(cfg, storage=storage, tile=tile)
            sim.set_tile(tile).set_grid_mode(mode).init(U).step(3)
            got = [sim.read_populations(k) for k in names]
            ref = ref or got
            assert all(torch.equal(a, b) for a, b in zip(ref, got)), (tile, mode)


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_persistent_grids_of_a_batch(storage):
    cfgs = [cfg_of(700 + 53 * i, 640 + 31 * i, 1, 1, 4) for i in range(5)]
    ref = None
    for tile in range(S.snowlb_tile_count()):
        tx, ty = tile_shape(tile)
        tiles = sum(-(-c["nx"] // tx) * -(-c["ny"] // ty) for c in cfgs)
        assert step_grid(tile, tiles, S.STORAGES[storage], 1, 1, 1) < tiles
        for mode in (0, 1, 3, 5):
            b = S.Batch(cfgs, storage).set_tile(tile, mode).init().step(3)
            got = [b.read(i, f) for i in range(len(cfgs)) for f in ("phi", "U", "rho", "ux", "uy")]
            ref = ref or got
            assert all(torch.equal(x, y) for x, y in zip(ref, got)), (tile, mode)
