"""Parameter gradients of the warm-start network for every width it has, against
the FP64 reference network, with the bar of the other gradient test: 1e-4 relative
per parameter array (float32 rounding through three layers); and for batches on
both sides of one element a block (up to 256 blocks), against the mean of the
gradients of its elements taken one at a time, with the same bar: the same
float32 terms, summed in another order.  (The reference itself is no help in
large batches: where an activation is within rounding of the relu's kink the
two sides take different branches, and some element of 64 has one.)
"""
import numpy as np
import pytest
import torch

from oracle import cnn
from synth.fields import make_field
from tests.test_gpu_cnn import _bf16, _element_kappa, _gpu_patches, _theta

pytestmark = pytest.mark.gpu


def _inputs(k, distinct):
    perm = make_field("gauss", 32, 7)
    kap = _element_kappa(perm)[:distinct] * 3.0 * 32 ** 2
    rng = np.random.default_rng(3)
    phis = [np.linalg.qr(rng.standard_normal((512, k)))[0] / np.sqrt(kap[e])[:, None] for e in range(distinct)]
    P, S = _gpu_patches(perm, 64)
    phi = torch.as_tensor(np.ascontiguousarray(np.stack([ph.T for ph in phis])), device="cuda")
    return perm, kap, phis, P.view(64, 1000)[:distinct], S.view(64, 512)[:distinct], phi


def _gradient(net, k, P, S, phi):
    count = P.shape[0]
    P, S, phi = P.contiguous(), S.contiguous(), phi.contiguous()
    X = torch.empty(count * net.kp * 512, dtype=torch.float32, device="cuda")
    net.forward(P, count, X)
    grad = torch.empty(net.n_params, dtype=torch.float32, device="cuda")
    loss = net.loss_backward(P, X, phi, k, S, count, grad)
    return loss, grad.cpu().numpy().astype(np.float64)


def _compare(k, a, b):
    off = 0
    for name, shp in cnn.param_shapes(k):
        size = int(np.prod(shp))
        x, y = a[off:off + size], b[off:off + size]
        assert np.linalg.norm(x - y) <= 1e-4 * np.linalg.norm(y), name
        off += size


@pytest.mark.parametrize("k,count", [(2, 1), (4, 3), (6, 2), (8, 5)])
def test_gradient_matches_oracle(k, count):
    from paper_2403_19342_amd.specmg import CNN
    perm, kap, phis, P, S, phi = _inputs(k, count)
    theta = _theta(2, k)
    net = CNN(k, count)
    net.load(torch.as_tensor(theta, device="cuda"))
    loss, g = _gradient(net, k, P, S, phi)
    lo, go = cnn.batch_loss_and_grad(_bf16(theta).astype(np.float64), k, cnn.patches(perm)[:count], phis, list(kap))
    assert abs(loss - lo) <= 1e-5 * lo
    _compare(k, g, go)
    net.close()


@pytest.mark.parametrize("k,count", [(6, 256), (6, 257), (8, 515)])
def test_batch_is_the_mean_of_its_elements(k, count):
    from paper_2403_19342_amd.specmg import CNN
    distinct = 8
    _, _, _, P, S, phi = _inputs(k, distinct)
    net = CNN(k, count)
    net.load(torch.as_tensor(_theta(2, k), device="cuda"))
    ones = [_gradient(net, k, P[e:e + 1], S[e:e + 1], phi[e:e + 1]) for e in range(distinct)]
    idx = torch.arange(count, device="cuda") % distinct
    loss, g = _gradient(net, k, P[idx], S[idx], phi[idx])
    order = [e % distinct for e in range(count)]
    assert abs(loss - np.mean([ones[e][0] for e in order])) <= 1e-6 * loss
    _compare(k, g, sum(ones[e][1] for e in order) / count)
    net.close()
