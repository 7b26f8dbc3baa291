"""Sizes at the edges of the dispatch rules: diagnostics of interfaces of few
and of many chunks (256 nodes or 512 triangles each), the one-launch network
passes (rows of 32 samples, widths up to 256) and the population exchange
(1024 cells per workgroup), against the oracle or a round trip."""
import numpy as np
import pytest

import oracle as o
import workloads as wl
from helpers import gpu_run, gpu_solver
from oracle import mlp as ref


def _network(widths, batch):
    rng = np.random.default_rng(5)
    p = ref.init_params(widths, 7)
    return p, rng.uniform(-1, 1, (batch, widths[0])), 0.3 * rng.standard_normal((batch, widths[-1]))


def _check_network(widths, p, x, t, y, loss, g):
    # bf16 operands, fp32 sums: the tolerances of the other network tests
    yo, _ = ref.forward(p, widths, x)
    lo, go = ref.loss_and_grad(p, widths, x, t)
    assert np.max(np.abs(y - yo)) <= 3e-2 * np.max(np.abs(yo))
    assert abs(loss - lo) <= 2e-2 * lo
    cos = float(np.dot(g, go) / (np.linalg.norm(g) * np.linalg.norm(go)))
    assert cos >= 0.999 and np.linalg.norm(g - go) <= 2e-2 * np.linalg.norm(go)


@pytest.mark.parametrize("widths,batch", [([4, 100, 5], 1), ([3, 256, 33], 33), ([4, 257, 40], 31)])
def test_network_edges_on_the_cpu(widths, batch):
    from emu import run_mlp
    p, x, t = _network(widths, batch)
    y, g, loss, _ = run_mlp(widths, p, x, t)
    _check_network(widths, p, x, t, y, loss, g)


@pytest.mark.gpu
@pytest.mark.parametrize("widths,batch", [([4, 100, 5], 1), ([4, 256, 256, 1281], 31), ([4, 64, 256, 33], 33),
                                          ([4, 257, 40], 33), ([4, 200, 100, 100], 4097)])
def test_network_edges(widths, batch):
    from paper_2503_20605_amd import MLP
    p, x, t = _network(widths, batch)
    print("[edges] network", widths, batch, flush=True)
    m = MLP(widths, batch)
    m.set_params(p)
    y = m.forward(x).cpu().numpy()
    loss, g = m.gradients(x, t)
    _check_network(widths, p, x, t, y, loss, g)


@pytest.mark.gpu
@pytest.mark.parametrize("nodes", [255, 257, 1024, 1025, 2600])
def test_diagnostics_2d_of_few_and_many_chunks(nodes):
    p = wl.Params(dim=2, nx=96, ny=40, tau=0.9, sigma=0.004, theta_eq_deg=70.0, xi=2.0)
    print("[edges] diagnostics 2D", nodes, flush=True)
    g = gpu_run(p, wl.cap_polygon(14.0, 90.0, 2.0, nodes, 48.0), 3)
    _check_diagnostics(2, g, None, p)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [6, 12])  # 720 and 2 880 triangles
def test_diagnostics_3d_of_few_and_many_chunks(n):
    p = wl.Params(dim=3, nx=48, ny=44, nz=24, bc=(0, 0, 1), tau=0.9, sigma=0.004, theta_eq_deg=70.0, xi=2.0)
    V, T = wl.cap_mesh(10.0, 90.0, 2.0, n, (24.0, 22.0))
    print("[edges] diagnostics 3D", len(V), len(T), flush=True)
    g = gpu_run(p, V, 2, tris=T)
    _check_diagnostics(3, g, T, p)


def _check_diagnostics(dim, g, tris, p):
    """From the state that is read back: double precision on both sides, only
    the order of the sums differs (fp32 fields enter the force sums exactly)."""
    d, q = g["solver"].diagnostics(0), g["q"]
    h = q[:, dim - 1]
    want = dict(volume=o.volume_2d(q) if dim == 2 else o.volume_3d(q, tris),
                contact_radius=o.contact_radius_2d(q, o.h_star(p.xi)) if dim == 2
                else o.contact_radius_3d(q, tris, o.h_star(p.xi)),
                height=h.max() - h.min(), min_h=h.min())
    e = (np.stack([np.arange(len(q)), np.roll(np.arange(len(q)), -1)], 1) if dim == 2
         else np.concatenate([tris[:, [0, 1]], tris[:, [1, 2]], tris[:, [2, 0]]]))
    el = np.linalg.norm(q[e[:, 1]] - q[e[:, 0]], axis=1)
    want.update(edge_min=el.min(), edge_max=el.max(), max_speed=np.linalg.norm(g["qdot"], axis=1).max())
    for k, v in want.items():
        assert abs(d[k] - v) <= 1e-11 * abs(v), k
    phi = g["phi"]
    assert np.max(np.abs(np.asarray(d["sum_phi"]) - phi.sum(0))) <= 1e-12 * np.abs(phi).sum()


@pytest.mark.gpu
@pytest.mark.parametrize("dim,nx,ny,nz", [(2, 31, 33, 1), (2, 1024, 1, 1), (2, 1025, 3, 1), (3, 5, 41, 3),
                                          (3, 32, 32, 2), (3, 41, 25, 65)])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_population_exchange_round_trip(dim, nx, ny, nz, storage):
    Q = 9 if dim == 2 else 19
    p = wl.Params(dim=dim, nx=nx, ny=ny, nz=nz, bc=(0, 0, 0), wetting=False)
    print("[edges] exchange", nx, ny, nz, storage, flush=True)
    # multiples of 2^-10 below 2^-3: exact in every storage
    f = np.random.default_rng(2).integers(-127, 128, (Q, nz, ny, nx)) / 1024.0
    s = gpu_solver([p], storage=storage)
    s.write_populations(0, f)
    assert np.array_equal(s.read_populations(0).cpu().numpy(), f)
