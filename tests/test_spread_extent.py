"""Spreading chunks (k_spread3) whose vertices fly apart or are not finite: the
box of cells that their taps cover is not formed from extents whose product
would overflow, and no index comes of it.  Runs in the sanitizer build only."""
import numpy as np
import pytest

import workloads as wl
from emu import run_case
from helpers import weights

C = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1]])


def _jump(p, u, where):
    """Populations that give the cells of `where` the velocity (u, u, u):
    momentum in the three axis pairs only."""
    f = np.zeros((19, p.nz, p.ny, p.nx))
    for i, c in enumerate(C):
        f[i][where] = 0.5 * u * c.sum()
    return f


@pytest.mark.parametrize("u", [4e6, 1.2e7, np.nan])
def test_vertices_far_apart_and_not_finite(u):
    p = wl.Params(dim=3, nx=20, ny=18, nz=16, bc=(0, 0, 0), tau=0.9, sigma=0.005, wetting=False)
    assert np.allclose(weights(3)[1:7], weights(3)[1])  # the axis directions come first
    V, T = wl.sphere_mesh(5.0, 3, (10.0, 9.0, 8.0))
    where = np.zeros((p.nz, p.ny, p.nx), bool)
    where[:, :, : 10 if np.isfinite(u) else 20] = True  # half of the vertices jump; all are NaN
    out = run_case([p], [V], [T], steps=(1, 2), f0dev=[_jump(p, u, where)])[0]
    # the first step reports the speed; a second one would spread from there
    assert out["status"] == -4
    out = run_case([p], [V], [T], steps=(4,), graph_steps=0, f0dev=[_jump(p, u, where)])[0]
    assert out["status"] == -4 and out["diag"]["status"] == -4


@pytest.mark.parametrize("far", [4e6, 1e12, 1e200])
def test_interface_set_with_vertices_far_apart(far):
    p = wl.Params(dim=3, nx=20, ny=18, nz=16, bc=(0, 0, 0), tau=0.9, sigma=0.005, wetting=False)
    V, T = wl.sphere_mesh(5.0, 3, (10.0, 9.0, 8.0))
    V = V.copy()
    V[::3] += far
    out = run_case([p], [V], [T], steps=(2,))[0]
    # beyond 2^24 a vertex is reported; up to there its taps wrap
    assert out["status"] == -4 or far < 2.0 ** 24
