"""Forward passes whose input and output share memory (same buffer, or
shifted against each other): equal, bit for bit, to the pass with separate
buffers."""
import ctypes

import numpy as np
import pytest

from oracle import mlp as ref

# one narrow network whose output columns are shared out among workgroups, one
# whose rows of input and output differ in length, one wide one
CASES = [([200, 256, 200], 40, 0, 0), ([200, 256, 200], 70, 0, 1000), ([100, 64, 300], 70, 500, 0),
         ([40, 300, 40], 40, 0, 0)]


def _network(widths, batch):
    rng = np.random.default_rng(6)
    return (ref.init_params(widths, 4), rng.uniform(-1, 1, (batch, widths[0])).astype(np.float32),
            np.zeros((batch, widths[-1]), np.float32))


@pytest.mark.parametrize("widths,batch,xoff,yoff", CASES)
def test_overlapping_forward_on_the_cpu(widths, batch, xoff, yoff):
    from emu import run_mlp
    p, x, t = _network(widths, batch)
    y, _, _, _, a, b = run_mlp(widths, p, x, t, overlap=(xoff, yoff))
    assert np.array_equal(y, a) and np.array_equal(y, b)


@pytest.mark.gpu
@pytest.mark.parametrize("widths,batch,xoff,yoff", CASES + [([200, 256, 200], 3300, 0, 0),
                                                            ([256, 256, 256], 2000, 0, 77)])
def test_overlapping_forward(widths, batch, xoff, yoff):
    import torch
    from paper_2503_20605_amd import MLP, _lib
    p, x, _ = _network(widths, batch)
    print("[overlap]", widths, batch, xoff, yoff, flush=True)
    m = MLP(widths, batch)
    m.set_params(p)
    y = m.forward(x).cpu().numpy()
    nx, ny = x.size, batch * widths[-1]
    for call in (m.lib.iblb_mlp_forward, m.lib.iblb_mlp_forward_noalloc):
        for _ in range(3):
            o = torch.zeros(max(xoff + nx, yoff + ny), dtype=torch.float32, device="cuda")
            o[xoff:xoff + nx] = torch.as_tensor(x.ravel()).cuda()
            torch.cuda.synchronize()
            _lib.check_mlp(call(m.h, ctypes.c_void_p(o.data_ptr() + 4 * xoff), batch,
                                ctypes.c_void_p(o.data_ptr() + 4 * yoff)), m.h)
            torch.cuda.synchronize()
            assert np.array_equal(o[yoff:yoff + ny].cpu().numpy().reshape(y.shape), y)
