"""The dense coarsest product at the ends of its range: 16 unknowns, both sides of
the row counts where a block takes more rows (1,024, 2,048), and 8,192, the most whose
right-hand side fits one LDS chunk.  With an exact coarsest solve on two levels
the preconditioner reproduces every function of the level-2 space it is given the
A-image of, up to the smoother: a solve then takes no more iterations than with
a third level over the same space, and reaches its tolerance.
"""
import pytest

from synth.fields import gaussian_log_field, make_source
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,eigs,unknowns", [((16, 8, 8), 8, 16), ((64, 32, 32), 8, 1024), ((64, 32, 40), 8, 1280),
                                                 ((64, 64, 32), 8, 2048), ((64, 64, 48), 8, 3072),
                                                 ((128, 64, 64), 8, 8192)])
def test_two_levels(shape, eigs, unknowns):
    import torch
    from paper_2403_19342_amd.specmg import SpecMG
    perm = to_dev(gaussian_log_field(64, 2, shape=shape))
    b = to_dev(make_source("corner", shape).reshape(-1))
    iters = {}
    for levels in (2, 3):
        if any(e % (8 * 2 ** (levels - 2)) for e in shape):
            continue
        ctx = SpecMG(perm, levels=levels, eigs_per_subdomain=eigs, agg=2, h=1.0 / 64)
        if levels == 2:
            assert ctx.info()["dims"][1] == unknowns
        x = torch.empty_like(b)
        rc, info = ctx.pcg_solve(b, x, tol=1e-9)
        assert rc == 0 and info.converged and info.rel_resid_true <= 1e-9
        iters[levels] = info.iters
        ctx.close()
    assert iters[2] <= iters.get(3, 1000) + 1
