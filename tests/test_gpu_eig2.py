"""Level-2 eigensolves at the edges of the block sizes (targets 1, 4, 5, 6, 7
and 8: blocks of 10, 12 and 14 columns, even and uneven shares per wavefront)
on elements that are hard for the small dense steps: homogeneous ones
(degenerate clusters, a cut inside a cluster), random values of contrast 1e8
(nearly dependent start columns), orthotropic; and a checkerboard of 2^3 cubes
of contrast 1e6, whose 32 nearly zero eigenvalues no block of 14 columns can
separate: set-up reports that.

Against the oracle's dense eigensolves: kept counts equal, kept eigenvalues
1e-11 (dimensionless, spectra in [0, 8]); the basis orthonormal in the weight
inner product to 1e-12 and its residual A phi - lambda S phi in the weighted
norm within 1e-11 of the spectral bound 8 (the stopping rule is 1e-12).
"""
import numpy as np
import pytest

from oracle import Grid, build_hierarchy
from oracle.assembly import element_cells, neumann_local
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _field(kind, shape):
    rng = np.random.default_rng(11)
    if kind == "homogeneous":
        return np.full(shape, 3.0)
    if kind == "checker":
        z, y, x = np.indices(shape)
        return np.where((x // 2 + y // 2 + z // 2) % 2 == 0, 1.0, 1.0e6)
    if kind == "ortho":
        return np.exp(rng.uniform(-4.0, 4.0, (3,) + shape))
    return np.exp(rng.uniform(-0.5 * np.log(1e8), 0.5 * np.log(1e8), shape))


@pytest.mark.parametrize("kind,target", [("homogeneous", 4), ("homogeneous", 8), ("random", 1), ("random", 4), ("random", 5),
                                         ("random", 6), ("random", 7), ("random", 8), ("ortho", 6)])
def test_level2_block_sizes(kind, target):
    from paper_2403_19342_amd.specmg import SpecMG
    shape = (8, 16, 24)
    perm = _field(kind, shape)
    nz, ny, nx = shape
    g = Grid(nx, ny, nz, 1.0 / nx, 1.0 / nx, 1.0 / nx)
    ref = build_hierarchy(perm, g, 2, target, sub=8, workers=1).level(2)
    ctx = SpecMG(to_dev(perm), levels=2, eigs_per_subdomain=target)
    lv = ctx.level_arrays(2)
    assert np.all(lv.status >= 0) and np.array_equal(lv.nkeep, ref.nkeep)
    kt = (perm if perm.ndim == 4 else np.stack([perm] * 3)) * nx ** 2
    cells = element_cells(g, (8, 8, 8))
    A = neumann_local(perm, g, (8, 8, 8)).tocsr()
    for e, k in enumerate(ref.nkeep):
        assert np.max(np.abs(lv.lam[e, :k] - ref.lam[e][:k])) < 1e-11
        S = kt.sum(0).reshape(-1)[cells[e]]
        phi = lv.basis[e, :k]
        assert np.max(np.abs((phi * S) @ phi.T - np.eye(k))) < 1e-12
        assert np.all(lv.basis[e, k:] == 0.0)
        Ae = A[cells[e]][:, cells[e]]
        res = (Ae @ phi.T - (S[:, None] * phi.T) * lv.lam[e, :k]) / np.sqrt(S)[:, None]
        assert np.max(np.linalg.norm(res, axis=0)) < 1e-11 * 8.0


@pytest.mark.parametrize("target", [1, 5])
def test_unresolvable_cluster_is_reported(target):
    from paper_2403_19342_amd.specmg import EEIG, SpecMG, SpecMGError
    with pytest.raises(SpecMGError) as e:
        SpecMG(to_dev(_field("checker", (8, 16, 24))), levels=2, eigs_per_subdomain=target)
    assert e.value.code == EEIG
