"""The coarse-coarse counts that a lower level's width admits with agg 4.

The eigensolver of a parent of 64 children keeps its block of vectors in one CU's
LDS, so the wide blocks (20 vectors for eigs_coarse 11..14, 26 for 15..20) need a
narrow lower level.  Set-up refuses what does not fit with EINVAL before it touches
the device; the widest that fit are set up and solve.
"""
import ctypes

import pytest

from synth.fields import make_field, make_source


def _refused(eigs, cc, levels=3, agg=4):
    from paper_2403_19342_amd.specmg import Grid, Opts, load_library
    lib = load_library()
    g = Grid(64, 64, 64, 1 / 64, 1 / 64, 1 / 64, 8, agg)
    o = Opts(levels, eigs, 1, 0, 0, None, 1e-12, 1e-6, 1e-3)
    o.eigs_coarse = cc
    o.eig_threshold = -1.0           # refused in any case, later and with another message
    ctx = ctypes.c_void_p()
    fake = ctypes.c_void_p(0x1000)   # never dereferenced: validation fails first
    rc = lib.specmg_setup(fake, 1, ctypes.byref(g), ctypes.byref(o), None, ctypes.byref(ctx))
    assert rc == -1 and ctx.value is None
    return "eigs_coarse" in lib.specmg_last_error().decode()


@pytest.mark.parametrize("eigs,cc,refused", [
    (8, 10, False), (7, 11, False), (8, 11, True), (7, 14, False), (8, 14, True), (2, 15, False), (3, 15, True),
    (2, 20, False), (3, 20, True), (8, 20, True)])
def test_block_too_large_is_refused_before_the_device(eigs, cc, refused):
    assert _refused(eigs, cc) == refused
    assert not _refused(eigs, cc, agg=2)
    assert not _refused(eigs, cc, levels=2)


@pytest.mark.gpu
@pytest.mark.parametrize("eigs,cc", [(8, 10), (7, 14), (2, 20)])
def test_widest_blocks_solve(eigs, cc):
    import torch
    from paper_2403_19342_amd.specmg import SpecMG
    from tests.gpu_util import to_dev
    perm = make_field("gauss", 64, 3)
    ctx = SpecMG(to_dev(perm), levels=3, eigs_per_subdomain=eigs, agg=4, eigs_coarse=cc)
    b = make_source("corner", perm.shape).reshape(-1)
    x = torch.empty(b.size, dtype=torch.float64, device="cuda")
    rc, info = ctx.pcg_solve(to_dev(b), x, tol=1e-9)
    assert rc == 0 and info.converged and info.rel_resid_true <= 1e-9 and info.eig_unconverged == 0
    ctx.close()
