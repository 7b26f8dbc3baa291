"""2D node kernel of batches with many nodes (k_ring2: pieces of up to 14
consecutive nodes): outlines at the edges of the pieces, one too coarse for
the box of cells in LDS, one across the periodic edge, with and without
re-spacing and two viscosities; one dense outline brings the batch to the
node count from which that kernel is used."""
import numpy as np
import pytest

import oracle as o
import workloads as wl
from emu import run_case
from helpers import collect, compare_fields, gpu_solver


def _batch():
    base = dict(dim=2, nx=44, ny=22, tau=0.9, sigma=0.005, theta_eq_deg=80.0, xi=2.0)
    ps, qs = [], []
    for n, R, xc, more in ((13, 5.0, 22.0, {}), (14, 14.0, 22.0, {}), (15, 6.0, 22.0, dict(respace=0.3)),
                           (28, 7.0, 22.0, {}), (29, 7.0, 2.0, dict(respace=0.2)), (43, 8.0, 22.0, dict(lam=3.0)),
                           (60, 8.0, 20.0, dict(bc=(1, 1, 0))), (5120, 8.0, 22.0, {})):
        ps.append(wl.Params(**base, **more))
        qs.append(wl.cap_polygon(R, 90.0, 2.0, n, xc))
    return ps, qs


def test_pieces_match_the_oracle_on_the_cpu():
    ps, qs = _batch()
    outs = run_case(ps, qs, steps=(2, 2), graph_steps=2)
    for d, (p, q) in enumerate(zip(ps, qs)):
        r = o.run(p, q, 4)
        drho, du, dq = compare_fields(outs[d], r, 2, f"pieces {len(q)}")
        assert outs[d]["status"] == 0
        assert drho <= 1e-6 and du <= 1e-5 and dq <= 1e-7


@pytest.mark.gpu
@pytest.mark.parametrize("storage", [0, 1])
def test_pieces_match_the_lone_droplet_bit_for_bit(storage):
    """The same droplets one by one take the kernel with 16 lanes per node."""
    ps, qs = _batch()
    print("[pieces] batch of", len(ps), flush=True)
    s = gpu_solver(ps, qs, storage=storage)
    s.set_graph_steps(16)
    s.step(41)
    for d in range(len(ps) - 1):
        one = gpu_solver([ps[d]], [qs[d]], storage=storage)
        one.step(41)
        a, b = collect(s, d, 2), collect(one, 0, 2)
        for k in ("rho", "U", "F", "fdev", "q", "qdot", "phi"):
            assert np.array_equal(a[k], b[k]), (len(qs[d]), k)
