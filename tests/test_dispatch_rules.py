"""Which kernels the rules of the dispatch pick at both sides of their lines, in
the sanitizer build, and what they give against the oracle."""
import numpy as np
import pytest

import oracle as o
import workloads as wl
from emu import run_case
from helpers import compare_fields
from oracle import mlp as ref


def _check_network(widths, batch, y, g, loss, x, t, p):
    # bf16 operands, fp32 sums: the tolerances of the other network tests
    yo, _ = ref.forward(p, widths, x)
    lo, go = ref.loss_and_grad(p, widths, x, t)
    assert np.max(np.abs(y - yo)) <= 3e-2 * np.max(np.abs(yo))
    assert abs(loss - lo) <= 2e-2 * lo
    cos = float(np.dot(g, go) / (np.linalg.norm(g) * np.linalg.norm(go)))
    assert cos >= 0.999 and np.linalg.norm(g - go) <= 2e-2 * np.linalg.norm(go)


def _network(widths, batch):
    rng = np.random.default_rng(5)
    return (ref.init_params(widths, 7), rng.uniform(-1, 1, (batch, widths[0])),
            0.3 * rng.standard_normal((batch, widths[-1])))


@pytest.mark.parametrize("nx,ny,nodes,ring", [(24, 16, [5119], False), (24, 16, [5120], True),
                                              (1400, 8, [5631], False), (1400, 8, [5632], True),
                                              (3000, 8, [8191], False), (3000, 8, [8192], True),
                                              (1400, 8, [5100, 19], False), (1400, 8, [5100, 20], True)])
def test_node_kernel_2d(nx, ny, nodes, ring):
    """k_ib_fused2 for few nodes, k_ring2 for many (a lone outline in a large
    box: later)."""
    p = wl.Params(dim=2, nx=nx, ny=ny, tau=0.9, sigma=0.005, theta_eq_deg=80.0, xi=2.0)
    qs = [wl.cap_polygon(4.0, 90.0, 2.0, n, nx / 2) for n in nodes]
    launches = []
    out = run_case([p] * len(nodes), qs, steps=(2,), launches=launches)
    assert any("k_ring2" in k for k in launches) == ring
    assert any("k_ib_fused2" in k for k in launches) != ring
    r = o.run(p, qs[-1], 2)
    drho, du, dq = compare_fields(out[-1], r, 2, f"nodes {nodes}")
    assert drho <= 1e-6 and du <= 1e-5 and dq <= 1e-7


# outline nodes or mesh frequency; diagnostics and contact radius by one
# workgroup or by several launches
@pytest.mark.parametrize("dim,size,diag_one,contact_one", [(2, 1280, True, True), (2, 1281, False, True),
                                                           (2, 5120, False, True), (2, 5121, False, False),
                                                           (3, 7, True, True), (3, 8, False, True),
                                                           (3, 11, False, True), (3, 12, False, False)])
def test_diagnostics_of_small_interfaces(dim, size, diag_one, contact_one):
    launches = []
    if dim == 2:
        p = wl.Params(dim=2, nx=24, ny=16, tau=0.9, sigma=0.005, theta_eq_deg=80.0, xi=2.0)
        q, t = wl.cap_polygon(6.0, 90.0, 2.0, size, 12.0), None
    else:
        p = wl.Params(dim=3, nx=20, ny=20, nz=12, bc=(0, 0, 1), tau=0.9, sigma=0.005, theta_eq_deg=80.0, xi=2.0)
        q, t = wl.cap_mesh(6.0, 90.0, 2.0, size, (10.0, 10.0))
    out = run_case([p], [q], [t], steps=(1,), contact=(3.0, 0.05), launches=launches)[0]
    assert any("k_diag_one" in k for k in launches) == diag_one
    assert any("k_diag_part" in k for k in launches) != diag_one
    assert any("k_contact_one" in k for k in launches) == contact_one
    assert any("k_contact_part" in k for k in launches) != contact_one
    # double precision on both sides, only the order of the sums differs
    want = o.contact_radius_2d(out["q"], 3.0) if dim == 2 else o.contact_radius_3d(out["q"], t, 3.0)
    assert abs(out["contact"][0] - want) <= 1e-11 * want
    want = o.volume_2d(out["q"]) if dim == 2 else o.volume_3d(out["q"], t)
    assert abs(out["diag"]["volume"] - want) <= 1e-11 * want


@pytest.mark.parametrize("nx,ny,nz", [(4, 4, 300), (3, 5, 200), (1, 1, 600), (16, 16, 9), (17, 16, 7), (40, 30, 5)])
def test_population_exchange_over_planes(nx, ny, nz):
    """Planes of less than a workgroup's lanes, of as many, of more: one step
    of the fluid from populations that differ in every element."""
    p = wl.Params(dim=3, nx=nx, ny=ny, nz=nz, bc=(0, 0, 1), tau=0.9, wetting=False)
    f = np.random.default_rng(8).uniform(-1e-3, 1e-3, (19, nz, ny, nx))
    out = run_case([p], steps=(1,), f0dev=[f])[0]
    w = o.lattice(3)[1][:, None, None, None]
    r = o.run(p, None, 1, f0=f + w)
    # fp32: the rounding of the input and of the collision
    assert np.max(np.abs(out["fdev"] - (r["f"] - w))) <= 1e-8


# narrow networks: many outputs for few rows, and a single layer, train layer
# by layer; the others in one launch
TRAINING = [([16, 24], 5, False), ([4, 24, 12000], 3, False), ([4, 24, 8000], 3, True), ([4, 16, 16, 70], 33, True),
            ([4, 300, 20], 3, False)]


@pytest.mark.parametrize("widths,batch,one", TRAINING)
def test_training_pass(widths, batch, one):
    from emu import run_mlp
    p, x, t = _network(widths, batch)
    launches = []
    y, g, loss, _ = run_mlp(widths, p, x, t, launches=launches)
    assert any("k_mlp_rows<1" in k for k in launches) == one
    assert any("k_mse_colsum" in k for k in launches) != one
    # the packed weights come with the update: set once, not packed again
    assert sum("k_pack" in k for k in launches) == (max(widths[:-1]) <= 256)
    _check_network(widths, batch, y, g, loss, x, t, p)


@pytest.mark.parametrize("widths", [[4, 8, 8, 2], [4, 32, 32, 32, 40], [4, 64, 64, 100]])
def test_workspace_of_narrow_layers(widths):
    """A row of the batch takes what a training pass keeps of it: per hidden
    layer the pre-activations (fp32, up to the next multiple of 32), per layer
    its input and its gradient (bf16); plus the loss sums."""
    import ctypes
    from paper_2503_20605_amd import _lib
    lib = _lib.load()
    W = (ctypes.c_int * len(widths))(*widths)
    size = [lib.iblb_mlp_workspace_bytes(len(widths) - 1, W, b) for b in (32000, 64000)]
    row = sum(4 * (-(-w // 32) * 32) for w in widths[1:-1]) + 2 * (sum(widths[:-1]) + sum(widths[1:])) + 1
    assert 0 < size[1] - size[0] <= 32000 * row


@pytest.mark.gpu
@pytest.mark.parametrize("widths,batch", [([4, 100, 33, 70], 40), ([256, 256, 1000], 33), ([20, 16384], 5), ([1, 1], 1)])
def test_updated_weights_are_the_ones_that_are_used(widths, batch):
    """After training steps the forward pass equals that of a network that was
    given the same weights, bit for bit."""
    from paper_2503_20605_amd import MLP
    p, x, t = _network(widths, batch)
    print("[rules] packed weights", widths, batch, flush=True)
    a, b = MLP(widths, batch), MLP(widths, batch)
    a.set_params(p)
    for _ in range(3):
        a.train_step(x, t, 1e-2)
    b.set_params(a.get_params())
    assert np.array_equal(a.forward(x).cpu().numpy(), b.forward(x).cpu().numpy())
    la, ga = a.gradients(x, t)
    lb, gb = b.gradients(x, t)
    assert la == lb and np.max(np.abs(ga - gb)) <= 1e-5 * np.max(np.abs(gb))  # (atomics: the order of the sums)


@pytest.mark.gpu
@pytest.mark.parametrize("widths,max_batch,batches", [([4, 64, 256, 16384], 1024, (1, 33, 512, 1024)),
                                                      ([16, 2000], 2400, (7, 2400)), ([200, 20], 64, (64,))])
def test_training_passes_of_one_network(widths, max_batch, batches):
    """Batches at both sides of the line on one handle, in turn."""
    from paper_2503_20605_amd import MLP
    p, _, _ = _network(widths, 1)
    m = MLP(widths, max_batch)
    m.set_params(p)
    for b in batches + batches[:1]:
        print("[rules] training", widths, b, flush=True)
        _, x, t = _network(widths, b)
        y = m.forward(x).cpu().numpy()
        loss, g = m.gradients(x, t)
        _check_network(widths, b, y, g, loss, x, t, p)
