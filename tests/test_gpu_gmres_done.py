"""GMRES queues the next direction's V-cycle before the host knows whether the step
before it converged; after the step that does, that V-cycle does no work.  The flag that
stops it is the context's, shared with CG: neither solver nor the preconditioner is
stopped by what another solve left in it.
"""
import numpy as np
import pytest

from synth.fields import make_field, make_source
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

SENTINEL = -7.25e-301


@pytest.mark.parametrize("precision,tol", [(0, 0.5), (0, 1e-3), (1, 1e-3), (2, 1e-3), (3, 1e-3)])
def test_no_v_cycle_after_the_last_step(monkeypatch, precision, tol):
    """The solver's vectors (V_0..V_k, Z_0..Z_{k-1}, w after k steps) lie in one buffer,
    here filled with a value that no vector holds."""
    import torch
    from paper_2403_19342_amd import specmg as sm
    held = {}

    def allocator():
        def alloc(nbytes, stream, user):
            t = torch.full(((nbytes + 7) // 8,), SENTINEL, dtype=torch.float64, device="cuda")
            held[t.data_ptr()] = t
            return t.data_ptr()

        fa, ff = sm._ALLOC_FN(alloc), sm._FREE_FN(lambda ptr, user: held.pop(ptr, None))
        return sm.Allocator(fa, ff, None), (fa, ff)

    monkeypatch.setattr(sm, "torch_allocator", allocator)
    perm = make_field("gauss", 32, 1)
    ctx = sm.SpecMG(to_dev(perm), levels=2, eigs_per_subdomain=4, agg=4, precision=precision)
    before = set(held)
    n, restart = perm.size, 20
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    rc, info = ctx.gmres_solve(to_dev(make_source("corner", perm.shape).reshape(-1)), x, restart=restart, tol=tol)
    torch.cuda.synchronize()
    assert rc == 0 and 1 <= info.iters < restart
    buf = max((held[a] for a in set(held) - before), key=lambda t: t.numel())
    vectors = to_host(buf)[:(2 * restart + 2) * n].reshape(-1, n)
    written = [bool((v != SENTINEL).any()) for v in vectors]
    assert sum(written) == 2 * info.iters + 2
    ctx.close()


def test_flag_is_not_left_for_the_next_call():
    import torch
    from paper_2403_19342_amd.specmg import SpecMG
    perm = to_dev(make_field("gauss", 32, 1))
    b = to_dev(make_source("corner", tuple(perm.shape)).reshape(-1))
    args = dict(levels=2, eigs_per_subdomain=4, agg=4)

    def calls(ctx):
        def solve(name, **kw):
            x = torch.zeros(b.numel(), dtype=torch.float64, device="cuda")
            rc, info = getattr(ctx, name)(b, x, tol=1e-8, raise_on_error=False, **kw)
            return to_host(x)

        def precond():
            z = torch.empty_like(b)
            ctx.apply_precond(b, z)
            return to_host(z)

        return {"gmres": lambda: solve("gmres_solve"), "pcg": lambda: solve("pcg_solve"), "precond": precond,
                "short gmres": lambda: solve("gmres_solve", max_iter=2)}

    alone = {}
    for name in ("gmres", "pcg", "precond", "short gmres"):
        ctx = SpecMG(perm, **args)
        alone[name] = calls(ctx)[name]()
        ctx.close()
    ctx = SpecMG(perm, **args)
    fs = calls(ctx)
    for name in ("gmres", "precond", "pcg", "gmres", "gmres", "pcg", "precond", "short gmres", "precond", "pcg"):
        assert np.array_equal(fs[name](), alone[name]), name
    ctx.close()
