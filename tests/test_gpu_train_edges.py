"""Gradient and training steps of the blend network at the edges of the
gradient kernel's split: chunks of 16 samples (one short, full, one over), as
many chunks as workgroups and one more, and a pair of training steps whose
second minibatch wraps.  Against the float64 oracle; the sums run in FP32 over
at most a few thousand products, so the bar is that of the oracle test of the
gradient, 1e-4 of its largest entry (1e-5 for the loss)."""
import numpy as np
import pytest
import torch

from oracle import mlp as M
from paper_2609_29081_amd import af

pytestmark = pytest.mark.gpu


def rows(n, seed):
    rng = np.random.default_rng(seed)
    X = 0.4 * rng.normal(size=(n, 40))
    y = np.clip(1.2 - rng.uniform(size=n) ** 2, 0.0, 1.0)
    p = 0.15 * rng.normal(size=M.NPARAM)
    return X.astype(np.float32), y.astype(np.float32), p.astype(np.float32)


def dev(*a):
    return [torch.as_tensor(z, device="cuda:0").contiguous() for z in a]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 16 * 256, 16 * 256 + 1, 16 * 700 + 5])
def test_gradient(n):
    X, y, p = rows(n, n)
    grad, loss = af.mlp_grad(*dev(X, y, p))
    lref, gref = M.loss_and_grad(*(a.astype(np.float64) for a in (p, X, y)))
    assert np.abs(grad.cpu().numpy() - gref).max() <= 1e-4 * np.abs(gref).max()
    assert abs(float(loss.item()) - lref) <= 1e-5 * lref


def test_training_equals_gradient_and_adam():
    """the fused update is the gradient call followed by the Adam call, bit
    for bit, minibatch by minibatch (the third wraps to the first row)"""
    X, y, p = rows(130, 3)
    Xd, yd, P = dev(X, y, p)
    m, v = torch.zeros_like(P), torch.zeros_like(P)
    P2, m2, v2 = P.clone(), m.clone(), v.clone()
    loss = af.mlp_train(Xd, yd, P, m, v, 4, 3, 50, 1e-3)
    for k, r in enumerate((0, 50, 0)):
        g, l2 = af.mlp_grad(Xd[r:r + 50].contiguous(), yd[r:r + 50].contiguous(), P2)
        af.mlp_adam(P2, g, m2, v2, 5 + k, 1e-3)
    assert torch.equal(P, P2) and torch.equal(m, m2) and torch.equal(v, v2)
    assert torch.equal(loss, l2)
