"""Thin Python binding of libsnowlb (include/snowlb.h).

Argument marshalling only: every step of the method runs in the HIP kernels of libsnowlb.  The
functions ``snowlb_*`` below carry the names and arguments of the C ABI; ``Sim`` is a convenience
object around one context that takes device memory and streams from PyTorch.  Importing this
module does not touch the GPU; loading the library fails loudly if it has not been built.  The
library is ``_lib/libsnowlb.so`` next to this file, or the file named by ``SNOWLB_LIB``.
"""
from __future__ import annotations

import ctypes
import os
from dataclasses import dataclass, fields

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("SNOWLB_LIB") or os.path.join(HERE, "_lib", "libsnowlb.so")

OK, EINVAL, ENOMEM, EDEVICE, EUNSUPPORTED, ENONFINITE, ESTATE = 0, -1, -2, -3, -4, -5, -6
STORE_FP32, STORE_FP16, STORE_BF16 = 0, 1, 2
BC_PERIODIC, BC_INOUT = 0, 1
FIELD_PHI, FIELD_U, FIELD_RHO, FIELD_UX, FIELD_UY = 0, 1, 2, 3, 4
POP_F, POP_G, POP_H, POP_PHIP = 0, 1, 2, 3
FIELDS = {"phi": FIELD_PHI, "U": FIELD_U, "rho": FIELD_RHO, "ux": FIELD_UX, "uy": FIELD_UY}
POPS = {"f": (POP_F, 9), "g": (POP_G, 5), "h": (POP_H, 9), "phip": (POP_PHIP, 1)}
STORAGES = {"fp32": STORE_FP32, "fp16": STORE_FP16, "bf16": STORE_BF16}


class SnowlbError(RuntimeError):
    def __init__(self, status: int, msg: str):
        super().__init__("%s: %s" % (_status_name(status), msg))
        self.status = status


class snowlb_params(ctypes.Structure):
    _fields_ = [
        ("nx", ctypes.c_int32), ("ny", ctypes.c_int32), ("flow", ctypes.c_int32),
        ("bc_x", ctypes.c_int32), ("storage", ctypes.c_int32), ("n_fold", ctypes.c_int32),
        ("eps", ctypes.c_double), ("W0", ctypes.c_double), ("tau0", ctypes.c_double),
        ("lam", ctypes.c_double), ("L_sat", ctypes.c_double), ("tau_vap", ctypes.c_double),
        ("tau_f", ctypes.c_double), ("h_drag", ctypes.c_double), ("kappa_N", ctypes.c_double),
        ("rho0", ctypes.c_double), ("u_in", ctypes.c_double), ("U_in", ctypes.c_double),
        ("grad_eps2", ctypes.c_double), ("U0", ctypes.c_double),
        ("seed_x", ctypes.c_double), ("seed_y", ctypes.c_double), ("seed_r", ctypes.c_double),
        ("init_width", ctypes.c_double), ("diag_every", ctypes.c_int32), ("tile", ctypes.c_int32),
        ("stencil", ctypes.c_int32), ("symmetric", ctypes.c_int32),
    ]


class snowlb3d_params(ctypes.Structure):
    _fields_ = [
        ("nx", ctypes.c_int32), ("ny", ctypes.c_int32), ("nz", ctypes.c_int32), ("flow", ctypes.c_int32),
        ("bc_x", ctypes.c_int32), ("diag_every", ctypes.c_int32),
        ("eps", ctypes.c_double), ("W0", ctypes.c_double), ("tau0", ctypes.c_double),
        ("lam", ctypes.c_double), ("L_sat", ctypes.c_double), ("tau_vap", ctypes.c_double),
        ("tau_f", ctypes.c_double), ("h_drag", ctypes.c_double), ("kappa_N", ctypes.c_double),
        ("rho0", ctypes.c_double), ("u_in", ctypes.c_double), ("U_in", ctypes.c_double),
        ("grad_eps2", ctypes.c_double), ("U0", ctypes.c_double),
        ("seed_x", ctypes.c_double), ("seed_y", ctypes.c_double), ("seed_z", ctypes.c_double),
        ("seed_r", ctypes.c_double), ("init_width", ctypes.c_double),
    ]


_lib = None

# exported symbol -> (restype, argtypes); the CPU-only ABI test checks this table against the headers
_P = ctypes.POINTER
_v = ctypes.c_void_p
_SIGS = {
    "snowlb_params_default": (None, [_P(snowlb_params)]),
    "snowlb_validate": (ctypes.c_int32, [_P(snowlb_params), _P(ctypes.c_char_p)]),
    "snowlb_status_str": (ctypes.c_char_p, [ctypes.c_int32]),
    "snowlb_last_error": (ctypes.c_char_p, [_v]),
    "snowlb_create": (ctypes.c_int32, [_P(snowlb_params), _P(_v)]),
    "snowlb_destroy": (None, [_v]),
    "snowlb_init": (ctypes.c_int32, [_v, _v, _v]),
    "snowlb_step": (ctypes.c_int32, [_v, ctypes.c_int32, _v]),
    "snowlb_step_count": (ctypes.c_int64, [_v]),
    "snowlb_read": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb_read_populations": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb_write_populations": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb_write_field": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb_diag": (ctypes.c_int32, [_v, _P(ctypes.c_double), _v]),
    "snowlb_diag_noalloc": (ctypes.c_int32, [_v, _v, _v]),
    "snowlb_state_bytes": (ctypes.c_int64, [_v]),
    "snowlb_save_state": (ctypes.c_int32, [_v, _v, ctypes.c_int64, _v]),
    "snowlb_load_state": (ctypes.c_int32, [_v, _v, ctypes.c_int64, _v]),
    "snowlb_tile_count": (ctypes.c_int32, []),
    "snowlb_tile_name": (ctypes.c_char_p, [ctypes.c_int32]),
    "snowlb_set_tile": (ctypes.c_int32, [_v, ctypes.c_int32]),
    "snowlb_get_tile": (ctypes.c_int32, [_v]),
    "snowlb_set_grid_mode": (ctypes.c_int32, [_v, ctypes.c_int32]),
    "snowlb_get_grid_mode": (ctypes.c_int32, [_v]),
    "snowlb_bw_probe": (ctypes.c_int32, [_v, _v, ctypes.c_int64, _v]),
    "snowlb_set_eps": (ctypes.c_int32, [_v, ctypes.c_double]),
    "snowlb_adj_forward": (ctypes.c_int32, [_v, ctypes.c_int32, ctypes.c_int32, _v]),
    "snowlb_adj_backward": (ctypes.c_int32, [_v, _v, _v, _P(ctypes.c_double), _P(ctypes.c_double), _v]),
    "snowlb_batch_create": (ctypes.c_int32, [_P(snowlb_params), ctypes.c_int32, _P(_v)]),
    "snowlb_batch_destroy": (None, [_v]),
    "snowlb_batch_size": (ctypes.c_int32, [_v]),
    "snowlb_batch_cells": (ctypes.c_int64, [_v]),
    "snowlb_batch_init": (ctypes.c_int32, [_v, _v]),
    "snowlb_batch_step": (ctypes.c_int32, [_v, ctypes.c_int32, _v]),
    "snowlb_batch_step_count": (ctypes.c_int64, [_v]),
    "snowlb_batch_read": (ctypes.c_int32, [_v, ctypes.c_int32, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb_batch_diag": (ctypes.c_int32, [_v, ctypes.c_int32, _P(ctypes.c_double), _v]),
    "snowlb_batch_set_tile": (ctypes.c_int32, [_v, ctypes.c_int32, ctypes.c_int32]),
    "snowlb_batch_get_tile": (ctypes.c_int32, [_v]),
    "snowlb_batch_last_error": (ctypes.c_char_p, [_v]),
    # three dimensions (include/snowlb3d.h)
    "snowlb3d_params_default": (None, [_P(snowlb3d_params)]),
    "snowlb3d_validate": (ctypes.c_int32, [_P(snowlb3d_params), _P(ctypes.c_char_p)]),
    "snowlb3d_create": (ctypes.c_int32, [_P(snowlb3d_params), _P(_v)]),
    "snowlb3d_destroy": (None, [_v]),
    "snowlb3d_last_error": (ctypes.c_char_p, [_v]),
    "snowlb3d_init": (ctypes.c_int32, [_v, _v, _v]),
    "snowlb3d_step": (ctypes.c_int32, [_v, ctypes.c_int32, _v]),
    "snowlb3d_step_count": (ctypes.c_int64, [_v]),
    "snowlb3d_read": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb3d_read_populations": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb3d_write_populations": (ctypes.c_int32, [_v, ctypes.c_int32, _v, ctypes.c_int64, _v]),
    "snowlb3d_diag": (ctypes.c_int32, [_v, _P(ctypes.c_double), _v]),
}


def lib():
    """Load libsnowlb.so (raises if it is missing: there is no fallback path)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("libsnowlb.so is not built (%s); run __graft_entry__.build() or "
                               "python -m paper_2101_07163_amd.build" % LIB_PATH)
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def _status_name(s: int) -> str:
    try:
        return lib().snowlb_status_str(s).decode()
    except Exception:  # pragma: no cover
        return "status %d" % s


def _check(status: int, ctx=None, batch=None, ctx3=False):
    if status != OK:
        if batch is not None:
            msg = lib().snowlb_batch_last_error(batch).decode()
        elif ctx3:
            msg = lib().snowlb3d_last_error(ctx).decode()
        else:
            msg = lib().snowlb_last_error(ctx).decode()
        raise SnowlbError(status, msg)


# ----------------------------------------------------------------------------- C-ABI, same names

def snowlb_params_default() -> snowlb_params:
    p = snowlb_params()
    lib().snowlb_params_default(ctypes.byref(p))
    return p


def snowlb_validate(p: snowlb_params) -> tuple[int, str]:
    msg = ctypes.c_char_p()
    s = lib().snowlb_validate(ctypes.byref(p), ctypes.byref(msg))
    return s, (msg.value or b"").decode()


def snowlb_create(p: snowlb_params) -> ctypes.c_void_p:
    ctx = ctypes.c_void_p()
    _check(lib().snowlb_create(ctypes.byref(p), ctypes.byref(ctx)), None)
    return ctx


def snowlb_destroy(ctx) -> None:
    lib().snowlb_destroy(ctx)


def snowlb_init(ctx, U_init_dev: int | None, stream: int) -> None:
    _check(lib().snowlb_init(ctx, U_init_dev, stream), ctx)


def snowlb_step(ctx, n: int, stream: int) -> None:
    _check(lib().snowlb_step(ctx, int(n), stream), ctx)


def snowlb_step_count(ctx) -> int:
    return int(lib().snowlb_step_count(ctx))


def snowlb_read(ctx, field: int, dst_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb_read(ctx, field, dst_dev, elems, stream), ctx)


def snowlb_read_populations(ctx, pset: int, dst_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb_read_populations(ctx, pset, dst_dev, elems, stream), ctx)


def snowlb_write_populations(ctx, pset: int, src_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb_write_populations(ctx, pset, src_dev, elems, stream), ctx)


def snowlb_write_field(ctx, field: int, src_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb_write_field(ctx, field, src_dev, elems, stream), ctx)


DIAG_COUNT = 9
DIAG_KEYS = ("rho", "jx", "jy", "U", "phi", "phi_prev", "n_solid", "n_nonfinite", "species")


def snowlb_diag(ctx, stream: int) -> tuple[int, list]:
    out = (ctypes.c_double * DIAG_COUNT)()
    s = lib().snowlb_diag(ctx, out, stream)
    if s not in (OK, ENONFINITE):
        _check(s, ctx)
    return s, list(out)


def snowlb_diag_noalloc(ctx, out_dev: int, stream: int) -> None:
    _check(lib().snowlb_diag_noalloc(ctx, out_dev, stream), ctx)


def snowlb_state_bytes(ctx) -> int:
    return int(lib().snowlb_state_bytes(ctx))


def snowlb_save_state(ctx, buf_dev: int, nbytes: int, stream: int) -> None:
    _check(lib().snowlb_save_state(ctx, buf_dev, nbytes, stream), ctx)


def snowlb_load_state(ctx, buf_dev: int, nbytes: int, stream: int) -> None:
    _check(lib().snowlb_load_state(ctx, buf_dev, nbytes, stream), ctx)


def snowlb_tile_count() -> int:
    return int(lib().snowlb_tile_count())


def snowlb_tile_name(i: int) -> str:
    return lib().snowlb_tile_name(i).decode()


def snowlb_set_tile(ctx, tile: int) -> None:
    _check(lib().snowlb_set_tile(ctx, tile), ctx)


def snowlb_get_tile(ctx) -> int:
    return int(lib().snowlb_get_tile(ctx))


def snowlb_set_grid_mode(ctx, mode: int) -> None:
    _check(lib().snowlb_set_grid_mode(ctx, mode), ctx)


def snowlb_get_grid_mode(ctx) -> int:
    return int(lib().snowlb_get_grid_mode(ctx))


def snowlb_bw_probe(dst_dev: int, src_dev: int, nbytes: int, stream: int) -> None:
    _check(lib().snowlb_bw_probe(dst_dev, src_dev, nbytes, stream), None)


def snowlb_set_eps(ctx, eps: float) -> None:
    _check(lib().snowlb_set_eps(ctx, float(eps)), ctx)


def snowlb_adj_forward(ctx, n_steps: int, ckpt_stride: int, stream: int) -> None:
    _check(lib().snowlb_adj_forward(ctx, int(n_steps), int(ckpt_stride), stream), ctx)


def snowlb_adj_backward(ctx, dL_dphiT_dev: int, dL_dUinit_dev: int, stream: int) -> tuple[float, float]:
    de, du = ctypes.c_double(), ctypes.c_double()
    _check(lib().snowlb_adj_backward(ctx, dL_dphiT_dev, dL_dUinit_dev, ctypes.byref(de), ctypes.byref(du),
                                     stream), ctx)
    return de.value, du.value


def snowlb_batch_create(params: list) -> ctypes.c_void_p:
    arr = (snowlb_params * len(params))(*params)
    b = ctypes.c_void_p()
    _check(lib().snowlb_batch_create(arr, len(params), ctypes.byref(b)), None)
    return b


def snowlb_batch_destroy(b) -> None:
    lib().snowlb_batch_destroy(b)


def snowlb_batch_size(b) -> int:
    return int(lib().snowlb_batch_size(b))


def snowlb_batch_cells(b) -> int:
    return int(lib().snowlb_batch_cells(b))


def snowlb_batch_init(b, stream: int) -> None:
    _check(lib().snowlb_batch_init(b, stream), batch=b)


def snowlb_batch_step(b, n: int, stream: int) -> None:
    _check(lib().snowlb_batch_step(b, int(n), stream), batch=b)


def snowlb_batch_step_count(b) -> int:
    return int(lib().snowlb_batch_step_count(b))


def snowlb_batch_read(b, i: int, field: int, dst_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb_batch_read(b, i, field, dst_dev, elems, stream), batch=b)


def snowlb_batch_diag(b, i: int, stream: int) -> tuple[int, list]:
    out = (ctypes.c_double * DIAG_COUNT)()
    s = lib().snowlb_batch_diag(b, i, out, stream)
    if s not in (OK, ENONFINITE):
        _check(s, batch=b)
    return s, list(out)


def snowlb_batch_set_tile(b, tile: int, grid_mode: int) -> None:
    _check(lib().snowlb_batch_set_tile(b, tile, grid_mode), batch=b)


def snowlb_batch_get_tile(b) -> int:
    return int(lib().snowlb_batch_get_tile(b))


# ----------------------------------------------------------------------------- convenience object

def make_params(cfg: dict, storage: str | int = "fp32", tile: int = 0, diag_every: int = 0) -> snowlb_params:
    """snowlb_params from a workload dict (keys as in workloads.py)."""
    p = snowlb_params_default()
    p.nx, p.ny = int(cfg["nx"]), int(cfg["ny"])
    p.flow = int(cfg.get("flow", 0))
    p.bc_x = int(cfg.get("inout", 0))
    p.storage = STORAGES[storage] if isinstance(storage, str) else int(storage)
    p.n_fold = int(cfg.get("n_fold", 6))
    p.stencil = int(cfg.get("stencil", 4))
    p.symmetric = int(cfg.get("symmetric", 0))
    for k in ("eps", "W0", "tau0", "lam", "L_sat", "tau_vap", "tau_f", "h_drag", "kappa_N", "rho0",
              "u_in", "U_in", "grad_eps2", "U0"):
        if k in cfg:
            setattr(p, k, float(cfg[k]))
    sx, sy, R = cfg.get("seed", (p.nx / 2, p.ny / 2, 5.0))
    p.seed_x, p.seed_y, p.seed_r = float(sx), float(sy), float(R)
    p.init_width = float(cfg.get("w_init", 1.0))
    p.tile = int(tile)
    p.diag_every = int(diag_every)
    return p


class Sim:
    """One lattice on the current GPU.  Buffers passed in and out are torch CUDA tensors."""

    def __init__(self, cfg: dict | snowlb_params, storage: str | int = "fp32", tile: int = 0,
                 diag_every: int = 0):
        import torch
        self.torch = torch
        self.p = cfg if isinstance(cfg, snowlb_params) else make_params(cfg, storage, tile, diag_every)
        self.ctx = snowlb_create(self.p)

    def __del__(self):
        ctx = getattr(self, "ctx", None)
        if ctx:
            try:
                snowlb_destroy(ctx)
            except Exception:  # interpreter shutdown: module globals may already be gone
                pass
            self.ctx = None

    @property
    def stream(self) -> int:
        return self.torch.cuda.current_stream().cuda_stream

    @property
    def shape(self):
        return (self.p.ny, self.p.nx)

    def init(self, U_init=None):
        ptr = None
        if U_init is not None:
            U_init = self.torch.as_tensor(U_init, dtype=self.torch.float32, device="cuda").contiguous()
            assert tuple(U_init.shape) == self.shape
            self._U_init = U_init  # keep alive until the kernel ran
            ptr = U_init.data_ptr()
        snowlb_init(self.ctx, ptr, self.stream)
        return self

    def step(self, n: int = 1):
        snowlb_step(self.ctx, n, self.stream)
        return self

    @property
    def step_count(self) -> int:
        return snowlb_step_count(self.ctx)

    def read(self, field: str):
        out = self.torch.empty(self.shape, dtype=self.torch.float32, device="cuda")
        snowlb_read(self.ctx, FIELDS[field], out.data_ptr(), out.numel(), self.stream)
        return out

    def read_populations(self, name: str):
        pset, q = POPS[name]
        out = self.torch.empty((q,) + self.shape, dtype=self.torch.float32, device="cuda")
        snowlb_read_populations(self.ctx, pset, out.data_ptr(), out.numel(), self.stream)
        return out if q > 1 else out[0]

    def write_field(self, field: str, values):
        """Overwrite phi (h = w phi, phi_prev = phi) or U (g at the equilibrium with the current velocity)."""
        t = self.torch.as_tensor(values, dtype=self.torch.float32, device="cuda").reshape(self.shape).contiguous()
        snowlb_write_field(self.ctx, FIELDS[field], t.data_ptr(), t.numel(), self.stream)
        self.torch.cuda.current_stream().synchronize()
        return self

    def write_populations(self, name: str, values):
        pset, q = POPS[name]
        t = self.torch.as_tensor(values, dtype=self.torch.float32, device="cuda").reshape(
            (q,) + self.shape).contiguous()
        snowlb_write_populations(self.ctx, pset, t.data_ptr(), t.numel(), self.stream)
        self.torch.cuda.current_stream().synchronize()
        return self

    def set_state(self, f=None, g=None, h=None, phip=None):
        # phi_prev first: with 16-bit storage h is encoded against it
        for name, v in (("phip", phip), ("f", f), ("g", g), ("h", h)):
            if v is not None:
                self.write_populations(name, v)
        return self

    def diag(self) -> dict:
        s, v = snowlb_diag(self.ctx, self.stream)
        d = dict(zip(DIAG_KEYS, v))
        d["status"] = s
        return d

    def save_state(self):
        n = snowlb_state_bytes(self.ctx)
        buf = self.torch.empty(n, dtype=self.torch.uint8, device="cuda")
        snowlb_save_state(self.ctx, buf.data_ptr(), n, self.stream)
        return buf

    def load_state(self, buf):
        snowlb_load_state(self.ctx, buf.data_ptr(), buf.numel(), self.stream)
        return self

    def set_tile(self, tile: int):
        snowlb_set_tile(self.ctx, tile)
        return self

    def set_grid_mode(self, mode: int):
        snowlb_set_grid_mode(self.ctx, mode)
        return self

    @property
    def tile(self) -> int:
        return snowlb_get_tile(self.ctx)

    @property
    def grid_mode(self) -> int:
        return snowlb_get_grid_mode(self.ctx)


class Batch:
    """Many independent lattices advanced by one launch per step (see snowlb_batch_* in the header)."""

    def __init__(self, cfgs: list, storage: str | int = "fp32", tile: int = 0):
        import torch
        self.torch = torch
        self.params = [c if isinstance(c, snowlb_params) else make_params(c, storage, tile) for c in cfgs]
        self.b = snowlb_batch_create(self.params)

    def __del__(self):
        b = getattr(self, "b", None)
        if b:
            try:
                snowlb_batch_destroy(b)
            except Exception:  # interpreter shutdown
                pass
            self.b = None

    @property
    def stream(self) -> int:
        return self.torch.cuda.current_stream().cuda_stream

    def __len__(self):
        return snowlb_batch_size(self.b)

    @property
    def cells(self) -> int:
        return snowlb_batch_cells(self.b)

    def init(self):
        snowlb_batch_init(self.b, self.stream)
        return self

    def step(self, n: int = 1):
        snowlb_batch_step(self.b, n, self.stream)
        return self

    @property
    def step_count(self) -> int:
        return snowlb_batch_step_count(self.b)

    def read(self, i: int, field: str):
        p = self.params[i]
        out = self.torch.empty((p.ny, p.nx), dtype=self.torch.float32, device="cuda")
        snowlb_batch_read(self.b, i, FIELDS[field], out.data_ptr(), out.numel(), self.stream)
        return out

    def diag(self, i: int) -> dict:
        s, v = snowlb_batch_diag(self.b, i, self.stream)
        d = dict(zip(DIAG_KEYS, v))
        d["status"] = s
        return d

    def set_tile(self, tile: int, grid_mode: int = 0):
        snowlb_batch_set_tile(self.b, tile, grid_mode)
        return self

    @property
    def tile(self) -> int:
        return snowlb_batch_get_tile(self.b)


def _adjoint_function():
    import torch

    class SnowAdjoint(torch.autograd.Function):
        """phi_T = SnowAdjoint.apply(eps, U_init, sim, n_steps, ckpt_stride).

        Forward: set eps, initialise the context `sim` (no flow, periodic, FP32) with the initial
        supersaturation field U_init, run n_steps with checkpoints every ckpt_stride steps (0: every state is
        kept while the states fit in the budget SNOWLB_ADJ_KEEP_MIB, 16 GiB by default for all contexts together, and in
        a quarter of the free memory; else sqrt(n_steps)).
        Backward: the library's hand-written adjoint gives dL/deps and dL/dU_init from dL/dphi_T;
        gradients with respect to anything U_init was built from (e.g. U0) follow by autograd.
        """

        @staticmethod
        def forward(ctx, eps, U_init, sim, n_steps, ckpt_stride=0):
            snowlb_set_eps(sim.ctx, float(eps))
            sim.init(U_init.detach())
            snowlb_adj_forward(sim.ctx, int(n_steps), int(ckpt_stride), sim.stream)
            ctx.sim = sim
            ctx.eps_like = eps
            return sim.read("phi")

        @staticmethod
        def backward(ctx, grad_phi):
            sim = ctx.sim
            g = grad_phi.detach().to(torch.float32).contiguous()
            dU = torch.empty_like(g)
            de, _ = snowlb_adj_backward(sim.ctx, g.data_ptr(), dU.data_ptr(), sim.stream)
            d_eps = torch.as_tensor(de, dtype=ctx.eps_like.dtype, device=ctx.eps_like.device)
            return d_eps, dU, None, None, None

    return SnowAdjoint


_SNOW_ADJOINT = None


def snow_adjoint(eps, U_init, sim: Sim, n_steps: int, ckpt_stride: int = 0):
    """Differentiable phi_T(eps, U_init) through the library's discrete adjoint (see SnowAdjoint)."""
    global _SNOW_ADJOINT
    if _SNOW_ADJOINT is None:
        _SNOW_ADJOINT = _adjoint_function()
    return _SNOW_ADJOINT.apply(eps, U_init, sim, n_steps, ckpt_stride)


# ----------------------------------------------------------------------------- three dimensions

FIELDS3 = {"phi": 0, "U": 1, "rho": 2, "ux": 3, "uy": 4, "uz": 5}
POPS3 = {"f": (POP_F, 19), "g": (POP_G, 7), "h": (POP_H, 7), "phip": (POP_PHIP, 1)}
DIAG3_KEYS = ("rho", "jx", "jy", "jz", "U", "phi", "phi_prev", "n_solid", "n_nonfinite", "species")


def snowlb3d_params_default() -> snowlb3d_params:
    p = snowlb3d_params()
    lib().snowlb3d_params_default(ctypes.byref(p))
    return p


def snowlb3d_validate(p: snowlb3d_params) -> tuple[int, str]:
    msg = ctypes.c_char_p()
    st = lib().snowlb3d_validate(ctypes.byref(p), ctypes.byref(msg))
    return st, (msg.value or b"").decode()


def snowlb3d_create(p: snowlb3d_params) -> ctypes.c_void_p:
    ctx = ctypes.c_void_p()
    _check(lib().snowlb3d_create(ctypes.byref(p), ctypes.byref(ctx)), None, ctx3=True)
    return ctx


def snowlb3d_destroy(ctx) -> None:
    lib().snowlb3d_destroy(ctx)


def snowlb3d_init(ctx, U_init_dev: int | None, stream: int) -> None:
    _check(lib().snowlb3d_init(ctx, U_init_dev, stream), ctx, ctx3=True)


def snowlb3d_step(ctx, n: int, stream: int) -> None:
    _check(lib().snowlb3d_step(ctx, int(n), stream), ctx, ctx3=True)


def snowlb3d_step_count(ctx) -> int:
    return int(lib().snowlb3d_step_count(ctx))


def snowlb3d_read(ctx, field: int, dst_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb3d_read(ctx, field, dst_dev, elems, stream), ctx, ctx3=True)


def snowlb3d_read_populations(ctx, pset: int, dst_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb3d_read_populations(ctx, pset, dst_dev, elems, stream), ctx, ctx3=True)


def snowlb3d_write_populations(ctx, pset: int, src_dev: int, elems: int, stream: int) -> None:
    _check(lib().snowlb3d_write_populations(ctx, pset, src_dev, elems, stream), ctx, ctx3=True)


def snowlb3d_diag(ctx, stream: int) -> tuple[int, list]:
    out = (ctypes.c_double * len(DIAG3_KEYS))()
    st = lib().snowlb3d_diag(ctx, out, stream)
    if st not in (OK, ENONFINITE):
        _check(st, ctx, ctx3=True)
    return st, list(out)


def make_params3d(cfg: dict, diag_every: int = 0) -> snowlb3d_params:
    """snowlb3d_params from a workload dict (keys as in workloads.py, seed = (x, y, z, R))."""
    p = snowlb3d_params_default()
    p.nx, p.ny, p.nz = int(cfg["nx"]), int(cfg["ny"]), int(cfg["nz"])
    p.flow = int(cfg.get("flow", 0))
    p.bc_x = int(cfg.get("inout", 0))
    for k in ("eps", "W0", "tau0", "lam", "L_sat", "tau_vap", "tau_f", "h_drag", "kappa_N", "rho0",
              "u_in", "U_in", "grad_eps2", "U0"):
        if k in cfg:
            setattr(p, k, float(cfg[k]))
    sx, sy, sz, R = cfg.get("seed", (p.nx / 2, p.ny / 2, p.nz / 2, 5.0))
    p.seed_x, p.seed_y, p.seed_z, p.seed_r = float(sx), float(sy), float(sz), float(R)
    p.init_width = float(cfg.get("w_init", 1.0))
    p.diag_every = int(diag_every)
    return p


class Sim3D:
    """One 3D lattice on the current GPU; buffers in and out are torch CUDA tensors ([z, y, x] fields)."""

    def __init__(self, cfg: dict | snowlb3d_params, diag_every: int = 0):
        import torch
        self.torch = torch
        self.p = cfg if isinstance(cfg, snowlb3d_params) else make_params3d(cfg, diag_every)
        self.ctx = snowlb3d_create(self.p)

    def __del__(self):
        ctx = getattr(self, "ctx", None)
        if ctx:
            try:
                snowlb3d_destroy(ctx)
            except Exception:  # interpreter shutdown
                pass
            self.ctx = None

    @property
    def stream(self) -> int:
        return self.torch.cuda.current_stream().cuda_stream

    @property
    def shape(self):
        return (self.p.nz, self.p.ny, self.p.nx)

    def init(self, U_init=None):
        ptr = None
        if U_init is not None:
            U_init = self.torch.as_tensor(U_init, dtype=self.torch.float32, device="cuda").contiguous()
            assert tuple(U_init.shape) == self.shape
            self._U_init = U_init
            ptr = U_init.data_ptr()
        snowlb3d_init(self.ctx, ptr, self.stream)
        return self

    def step(self, n: int = 1):
        snowlb3d_step(self.ctx, n, self.stream)
        return self

    @property
    def step_count(self) -> int:
        return snowlb3d_step_count(self.ctx)

    def read(self, field: str):
        out = self.torch.empty(self.shape, dtype=self.torch.float32, device="cuda")
        snowlb3d_read(self.ctx, FIELDS3[field], out.data_ptr(), out.numel(), self.stream)
        return out

    def read_populations(self, name: str):
        pset, q = POPS3[name]
        out = self.torch.empty((q,) + self.shape, dtype=self.torch.float32, device="cuda")
        snowlb3d_read_populations(self.ctx, pset, out.data_ptr(), out.numel(), self.stream)
        return out if q > 1 else out[0]

    def write_populations(self, name: str, values):
        pset, q = POPS3[name]
        t = self.torch.as_tensor(values, dtype=self.torch.float32, device="cuda").reshape((q,) + self.shape).contiguous()
        snowlb3d_write_populations(self.ctx, pset, t.data_ptr(), t.numel(), self.stream)
        self.torch.cuda.current_stream().synchronize()
        return self

    def set_state(self, f=None, g=None, h=None, phip=None):
        for name, v in (("phip", phip), ("f", f), ("g", g), ("h", h)):
            if v is not None:
                self.write_populations(name, v)
        return self

    def diag(self) -> dict:
        st, v = snowlb3d_diag(self.ctx, self.stream)
        d = dict(zip(DIAG3_KEYS, v))
        d["status"] = st
        return d
