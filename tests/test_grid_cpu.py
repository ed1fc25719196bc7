"""The wavelength grid's check on the host: what the rule on the log10 steps
accepts and refuses, the library's quicker first look included."""

import ctypes

import numpy as np
import pytest

from paper_2512_24840_amd import lasp


def accepted(grid):
    o = lasp.LaspOpts()
    lasp.load().lasp_default_opts(ctypes.byref(o))
    o.n_spec, o.n_pix = 1, grid.size
    g = np.ascontiguousarray(grid)
    return lasp.load().lasp_pool_slot_bytes(ctypes.byref(o), g.ctypes.data_as(ctypes.c_void_p)) > 0


def rule(w):
    with np.errstate(all="ignore"):
        if not np.all((w > 0) & np.isfinite(w)):
            return False
        dl = np.log10(w[-1] / w[0]) / (w.size - 1)
        return bool(dl > 0 and not np.any(np.abs(np.log10(w[1:] / w[:-1]) - dl) > 1e-6 * dl))


@pytest.mark.parametrize("n", [32, 33, 1550, 8000])
@pytest.mark.parametrize("step", [1e-3, 1e-4, 5.58e-5, 1e-7])
def test_grids_beside_the_tolerance(n, step):
    if n * step > 3:
        pytest.skip("outside any wavelength range")
    for lam0 in (1e-300, 3700.0, 1e300):
        base = lam0 * 10.0 ** (step * np.arange(n))
        assert accepted(base) == rule(base)
        for rel in (0.5, 0.9, 0.999, 1.001, 1.1, 2.0, 100.0):
            for j in (0, 1, n // 2, n - 2, n - 1):
                for sign in (1.0, -1.0):
                    w = base.copy()
                    w[j] *= 10.0 ** (sign * rel * 1e-6 * step)
                    assert accepted(w) == rule(w), (lam0, rel, j, sign)


def test_what_is_no_grid():
    base = 3700.0 * 10.0 ** (1e-4 * np.arange(64))
    for j in (0, 5, 63):
        for v in (0.0, -1.0, np.nan, np.inf, -np.inf, 1e308, 5e-324):
            w = base.copy()
            w[j] = v
            assert accepted(w) == rule(w), (j, v)
    assert not accepted(base[::-1])
    assert not accepted(np.full(64, 5000.0))
    assert not accepted(np.linspace(3700.0, 3800.0, 64))
    tiny = 5000.0 * (1.0 + 1e-15 * np.arange(64))       # steps of a few last bits
    assert accepted(tiny) == rule(tiny)
