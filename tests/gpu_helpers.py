"""Shared helpers of the GPU parity tests (tolerances, error metrics, input staging)."""
import ctypes
import sys

import numpy as np
import torch

import paper_2609_34972_amd as dvl

# Parity bar: normwise max relative error ||x - ref||_inf / ||ref||_inf per output
# tensor (and per layer), 1e-4 for fp32 runs and 2e-2 for bf16 runs.
TOL = {"f32": 1e-4, "bf16": 2e-2}


def say(*args):
    print(*args, flush=True)
    sys.stdout.flush()


def rel_err(x, ref) -> float:
    x = np.asarray(x, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    den = float(np.max(np.abs(ref)))
    num = float(np.max(np.abs(x - ref)))
    if den == 0.0:
        return num
    return num / den


def assert_close(x, ref, dtype: str, what: str):
    e = rel_err(x, ref)
    assert np.all(np.isfinite(np.asarray(x, dtype=np.float64))), f"{what}: non-finite output"
    assert e <= TOL[dtype], f"{what}: normwise relative error {e:.3e} > {TOL[dtype]:.0e}"
    return e


def f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to("cpu").to(torch.float64).numpy()


def cuda(t: torch.Tensor) -> torch.Tensor:
    return t.to("cuda:0").contiguous()


def launch_rule(name: str, restype, *args):
    """A launch rule of the library (a C++ function of namespace dv, by its mangled name), called on
    (ctypes type, value) pairs: tests that need a certain kernel assert that their sizes reach it."""
    f = getattr(dvl.load(), name)
    f.restype, f.argtypes = restype, [t for t, _ in args]
    return f(*(v for _, v in args))


# Tile shapes of the bf16 down projection (the library's DownTiles).
DOWN_DEEP, DOWN_256, DOWN_192, DOWN_128 = range(4)


def down_tiles(T: int, N: int) -> int:
    return launch_rule("_ZN2dv10down_tilesEll", ctypes.c_int, (ctypes.c_int64, T), (ctypes.c_int64, N))


def up_layers_per_block(T: int, d: int, nl: int) -> int:
    """Layers that a block of the tiled bf16 up projection takes in a launch of nl."""
    tiles = -(-T // 128) * -(-d // 128)
    return launch_rule("_ZN2dv19up_layers_per_blockEli", ctypes.c_int, (ctypes.c_int64, tiles), (ctypes.c_int, nl))
