"""The block smoother of a non-coarsest level whose width lies between the
instantiated ones (14 to 22), against the FP64 oracle: L_cc = 11, 12 and 16
at four levels with 2x aggregation, so that level 3 is 14, 15 and 19 wide.

Tolerances as in the other parity tests: P^{-1} r max(1e-10,
1e-15 / lambda_min+(A_L)) relative, PCG iterations within +-1, solution 1e-8.
"""
import numpy as np
import pytest

from oracle import Grid, build_hierarchy, Preconditioner, pcg
from synth.fields import make_field, make_source, random_zero_mean
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,seed,cc", [("inclusions", 3, 11), ("gauss", 1, 12), ("inclusions", 3, 16)])
def test_sweep_between_widths(kind, seed, cc):
    import torch
    from paper_2403_19342_amd.specmg import SpecMG
    n, levels, eigs = 64, 4, 6
    perm = make_field(kind, n, seed)
    g = Grid.unit_cube(n)
    hier = build_hierarchy(perm, g, levels, eigs, sub=8, agg=2, workers=8, target_cc=cc)
    ctx = SpecMG(to_dev(perm), levels=levels, eigs_per_subdomain=eigs, agg=2, eigs_coarse=cc)
    assert ctx.info()["widths"][2] == cc + 3
    pre = Preconditioner(hier)
    wL = np.linalg.eigvalsh(hier.level(levels).A.toarray())
    r = random_zero_mean(perm.shape, 300).reshape(-1)
    z = torch.empty(g.n, dtype=torch.float64, device="cuda")
    ctx.apply_precond(to_dev(r), z)
    zg, zo = to_host(z), pre.apply(r)
    zg -= zg.mean()
    zo -= zo.mean()
    err = np.linalg.norm(zg - zo) / np.linalg.norm(zo)
    print(f"{kind} L_cc {cc}: P^-1 r rel err {err:.2e}")
    assert err < max(1e-10, 1e-15 / wL[1])
    b = make_source("corner", perm.shape).reshape(-1)
    ref = pcg(hier.A, b, pre.apply, tol=1e-6)
    x = torch.empty(g.n, dtype=torch.float64, device="cuda")
    rc, info = ctx.pcg_solve(to_dev(b), x, tol=1e-6)
    assert rc == 0 and abs(info.iters - ref.iters) <= 1
    assert np.linalg.norm(to_host(x) - ref.x) <= 1e-8 * np.linalg.norm(ref.x)
