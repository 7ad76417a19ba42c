"""Flexible GMRES at restart lengths around the 16 and 32 basis vectors that the
projection keeps in registers (longer cycles go by passes), against the
oracle.  A weak preconditioner (two levels, one kept mode) makes the cycles long.

Bars of the other GMRES tests: Arnoldi steps and restarts within +-1, zero-mean
solutions within 1e-8 relative.  The system is solved to 1e-10, so that each side
is within about 1e-10 times the preconditioned condition number of the solution.
"""
import numpy as np
import pytest

from oracle import Grid, Preconditioner, build_hierarchy, fgmres
from synth.fields import make_field, make_source
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [15, 16, 17, 32, 33, 64])
def test_restart_lengths(restart):
    import torch
    from paper_2403_19342_amd.specmg import SpecMG
    perm = make_field("gauss", 32, 2)
    g = Grid.unit_cube(32)
    hier = build_hierarchy(perm, g, 2, 1, sub=8, agg=2, workers=1)
    b = make_source("corner", perm.shape).reshape(-1)
    ref = fgmres(hier.A, b, Preconditioner(hier).apply, tol=1e-10, restart=restart)
    ctx = SpecMG(to_dev(perm), levels=2, eigs_per_subdomain=1, agg=2)
    x = torch.empty(g.n, dtype=torch.float64, device="cuda")
    rc, info = ctx.gmres_solve(to_dev(b), x, restart=restart, tol=1e-10)
    xg = to_host(x)
    assert rc == 0 and info.converged and ref.converged
    assert abs(info.iters - ref.iters) <= 1
    assert abs(info.replacements - ref.restarts) <= 1
    assert np.linalg.norm(xg - ref.x) <= 1e-8 * np.linalg.norm(ref.x)
