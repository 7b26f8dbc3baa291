"""Cell sums over groups of several tiles, and the wall losses of the 2D node
kernel for many nodes."""
import numpy as np
import pytest

import oracle as o
import workloads as wl
from emu import run_case
from helpers import collect, gpu_solver


def _near_the_wall():
    """Outlines whose lower nodes lose taps to the wall; a dense one brings
    the batch to the node count of k_ring2."""
    base = dict(dim=2, nx=44, ny=22, tau=0.9, sigma=0.005, wetting=False)
    ps, qs = [], []
    for n, R, h, more in ((13, 5.0, 0.7, {}), (29, 7.0, 1.2, dict(respace=0.2)), (60, 8.0, 0.9, dict(bc=(1, 1, 0))),
                          (5120, 8.0, 2.0, {})):
        ps.append(wl.Params(**base, **more))
        qs.append(wl.cap_polygon(R, 90.0, h, n, 22.0))
    return ps, qs


def test_wall_losses_of_many_nodes_on_the_cpu():
    ps, qs = _near_the_wall()
    launches = []
    outs = run_case(ps, qs, steps=(3,), launches=launches)
    assert any("k_ring2" in k for k in launches) and not any("k_ib_fused2" in k for k in launches)
    for d in range(3):
        a = np.asarray(outs[d]["diag"]["dropped_F"])
        # fp32 forces and weights
        want = o.run(ps[d], qs[d], 3)["dropped"][:2]
        assert np.max(np.abs(a)) > 0
        assert np.max(np.abs(a - want)) <= 1e-5 * np.sum(np.abs(outs[d]["phi"]))


@pytest.mark.gpu
def test_wall_losses_of_many_nodes_match_the_lone_droplet():
    """k_ring2 against k_ib_fused2: the same bits (on the device, whose
    compiler fuses the products of the latter; not on the CPU)."""
    ps, qs = _near_the_wall()
    print("[sums] wall losses", flush=True)
    s = gpu_solver(ps, qs)
    s.step(9)
    batch = s.diagnostics(-1)
    for d in range(3):
        one = gpu_solver([ps[d]], [qs[d]])
        one.step(9)
        a, b = batch[d]["dropped_F"], one.diagnostics(0)["dropped_F"]
        assert a == b and np.max(np.abs(a)) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_cell_sums_over_groups_of_tiles(storage):
    """4x128x130 has 16 640 tiles, two to a group, and a last group of its own
    for the droplet that follows; mass, momentum and force against sums of the
    fields that are read back (double precision on both sides)."""
    big = wl.Params(dim=3, nx=4, ny=128, nz=130, bc=(0, 0, 1), tau=0.9, wetting=False)
    small = wl.Params(dim=3, nx=24, ny=21, nz=15, bc=(0, 0, 1), tau=0.9, sigma=0.005, theta_eq_deg=70.0, xi=2.0)
    V, T = wl.cap_mesh(6.0, 90.0, 2.0, 4, (12.0, 10.5))
    print("[sums] storage", storage, flush=True)
    s = gpu_solver([small, big, small], [V, None, V], [T, None, T], storage=storage)
    rng = np.random.default_rng(4)
    s.write_populations(1, rng.uniform(-1e-2, 1e-2, (19, 130, 128, 4)))
    F = rng.uniform(-1e-5, 1e-5, (3, 130, 128, 4)).astype(np.float32)
    s.set_force_field(1, F)
    s.step(3)
    for d, dg in enumerate(s.diagnostics(-1)):
        g = collect(s, d, 3)
        cells = g["rho"].size
        mass = cells + g["fdev"].sum()
        assert abs(dg["mass"] - mass) <= 1e-12 * cells
        for a in range(3):
            m, f = g["rho"] * g["U"][a], g["F"][a]
            assert abs(dg["momentum"][a] - m.sum()) <= 1e-11 * np.abs(m).sum()
            assert abs(dg["sum_F"][a] - f.sum()) <= 1e-11 * np.abs(f).sum()
        assert np.abs(g["F"]).sum() > 0 and np.abs(g["U"]).sum() > 0
