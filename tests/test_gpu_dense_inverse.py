"""The dense inverse of the coarsest matrix at the edges of its 64-wide blocks.

The kernels take any multiple of 32 rows; the elimination by blocks of 64 pads
an odd half block with the identity, and above 8192 rows panels of 256 columns
take over.  Reference: the matrix is built from its eigenvectors, so its inverse is
known.  Tolerance: the inverse from a Cholesky factor has a relative
error of at most a small multiple of n eps cond(A) (Higham, Accuracy and
Stability of Numerical Algorithms, ch. 14); 4 is used here.
"""
import ctypes

import pytest
import torch

from paper_2403_19342_amd.specmg import load_library

pytestmark = pytest.mark.gpu


def _inverse(a):
    lib = load_library()
    inverse = lib._ZN6specmg17dense_spd_inverseEPdiS0_S0_PiP12ihipStream_t
    inverse.restype = ctypes.c_int
    work_size = lib._ZN6specmg30dense_spd_inverse_work_doublesEi
    tbuf_size = lib._ZN6specmg30dense_spd_inverse_tbuf_doublesEi
    work_size.restype = tbuf_size.restype = ctypes.c_size_t
    n = a.shape[0]
    a = a.clone()
    work = torch.full((work_size(n),), float("nan"), dtype=torch.float64, device="cuda")
    tbuf = torch.full((tbuf_size(n),), float("nan"), dtype=torch.float64, device="cuda")
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    assert inverse(ptr(a), ctypes.c_int(n), ptr(work), ptr(tbuf), ptr(bad), ctypes.c_void_p(0)) == 0
    return a, int(bad.item())


def _reflect(x, v):
    return x - 2.0 * torch.outer(v, v @ x)


@pytest.mark.parametrize("n", [32, 64, 96, 160, 1024, 2080, 8192, 8224])
@pytest.mark.parametrize("cond", [1e2, 1e8])
def test_inverse_of_known_matrix(n, cond):
    g = torch.Generator().manual_seed(n)
    d = torch.logspace(0, float(torch.log10(torch.tensor(cond))), n, dtype=torch.float64)
    d = d[torch.randperm(n, generator=g)].cuda()
    vs = [torch.randn(n, generator=g, dtype=torch.float64).cuda() for _ in range(3)]
    a, ref = torch.diag(d), torch.diag(1.0 / d)
    for v in vs:   # A = Q D Q^T, Q a product of reflections
        v = v / v.norm()
        a, ref = _reflect(_reflect(a, v).T.contiguous(), v), _reflect(_reflect(ref, v).T.contiguous(), v)
    a = 0.5 * (a + a.T)
    x, bad = _inverse(a)
    assert bad == 0
    assert torch.equal(x, x.T)
    err = float((x - ref).norm() / ref.norm())
    assert err <= 4 * n * 2.0**-53 * cond


@pytest.mark.parametrize("n,row", [(64, 0), (96, 17), (160, 130)])
def test_a_negative_pivot_is_reported(n, row):
    a = torch.eye(n, dtype=torch.float64, device="cuda")
    a[row, row] = -1.0
    x, bad = _inverse(a)
    assert bad == 4
    assert torch.isfinite(x).all()
