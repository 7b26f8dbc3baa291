"""Spreading chunks (k_spread3) whose vertices fly apart or are not finite: the
box of cells that their taps cover is not formed from extents whose product
would overflow, and no index comes of it (in the sanitizer build only).  And
chunks that have outgrown the box: taken in runs, or added straight to memory,
they give the sums of chunks that fit."""
import numpy as np
import pytest

import workloads as wl
from emu import run_case, run_cases
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


@pytest.mark.parametrize("R,nu", [(10.0, 6), (13.0, 2), (3.0, 4)])
def test_outgrown_chunks_give_the_same_sums(R, nu):
    """One build cuts the chunks to the box, the other does not: 64 vertices
    of (10, 6) need more than 2 800 cells and half of their runs of 16 more than
    1536, all runs of (13, 2) do, (3, 4) fits as a whole.  Sums in
    fixed point: equal bit for bit."""
    p = wl.Params(dim=3, nx=34, ny=33, nz=32, bc=(0, 0, 0), tau=0.9, sigma=0.005, wetting=False)
    V, T = wl.sphere_mesh(R, nu, (17.0, 16.5, 16.0))
    a, b = run_cases([dict(params_list=[p], nodes_list=[V], tris_list=[T], steps=(2,), direct_chunks=k)
                      for k in (False, True)])
    for k in ("F", "U", "q", "phi"):
        assert np.array_equal(a[0][k], b[0][k]), k
    assert np.abs(a[0]["F"]).max() > 0


@pytest.mark.gpu
def test_outgrown_chunks_match_the_oracle():
    """A cap whose flat base a shear flow (u_z up to 0.1, varying along x)
    folds: its chunks are cut to 1200 cells at the start; after 60 steps 16 of
    46 have boxes of more than 1536, and so have some of their runs.  fp32
    against the FP64 oracle at the bounds of the other 3D parity tests."""
    import oracle as o
    from helpers import compare_fields, gpu_run
    p = wl.Params(dim=3, nx=48, ny=48, nz=40, bc=(0, 0, 0), tau=0.6, sigma=0.005, wetting=False)
    V, T = wl.cap_mesh(16.0, 90.0, 10.0, 12, (24.0, 24.0))
    c, w = o.lattice(3)
    uz = np.broadcast_to(0.1 * np.sin(2 * np.pi * (np.arange(48) + 0.5) / 24), (40, 48, 48))
    f = np.stack([3 * w[i] * c[i][2] * uz for i in range(19)])
    print("[outgrown]", len(V), flush=True)
    g = gpu_run(p, V, 60, tris=T, f0dev=f)
    r = o.run(p, V, 60, tris=T, f0=f + w[:, None, None, None])
    drho, du, dq = compare_fields(g, r, 3, "outgrown")
    assert drho <= 1e-5 and du <= 1e-5 and dq <= 1e-5
