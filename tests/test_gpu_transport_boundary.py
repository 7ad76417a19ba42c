"""The velocities of boundary faces are not read (the header's promise): an array that
ends before the last plane's, and the array of an axis of one cell, of which no
value is needed, give the result of full arrays to the bit.  The grids are larger than
what an allocator rounds a short array up to.
"""
import ctypes

import numpy as np
import pytest

from synth.fields import random_saturation
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1200, 1300), (1300, 1, 1200), (1200, 1300, 1), (2, 1200, 700), (7, 601, 400)])
def test_short_arrays(shape):
    import torch
    from paper_2403_19342_amd.specmg import Grid, load_library, transport
    rng = np.random.default_rng(shape[1])
    nz, ny, nx = shape
    h = (0.1, 0.05, 0.01)
    s0 = random_saturation(shape, 3)
    phi, q = to_dev(rng.uniform(0.05, 0.35, shape)), to_dev(rng.standard_normal(shape))
    v = [rng.standard_normal(shape) for _ in range(3)]
    work = torch.empty(2 * s0.size + 2048, dtype=torch.float64, device="cuda")
    t = torch.empty(1, dtype=torch.float64, device="cuda")
    full = to_dev(s0)
    transport(phi, q, *(to_dev(a) for a in v), full, h, 3, 1e-2, work, t)
    t_full = float(t)
    # x and y: everything up to the last interior face; z: the planes but the last
    used = [s0.size - 1 if nx > 1 else 1, s0.size - nx if ny > 1 else 1, s0.size - nx * ny if nz > 1 else 1]
    short = [to_dev(np.ascontiguousarray(a.reshape(-1)[:m])) for a, m in zip(v, used)]
    s = to_dev(s0)
    g = Grid(nx, ny, nz, *h, 8, 2)
    p = lambda a: ctypes.c_void_p(a.data_ptr())
    rc = load_library().specmg_transport(ctypes.byref(g), p(phi), p(q), p(short[0]), p(short[1]), p(short[2]), p(s), 3,
                                         1e-2, p(work), p(t), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    assert np.array_equal(to_host(s), to_host(full)) and float(t) == t_full
