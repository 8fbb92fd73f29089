"""Selector training and forward kernels at the edges of their sample tiles, against FP64."""
import numpy as np
import pytest

from oracle import mlp as omlp


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1, 15, 16, 17, 31, 32, 33, 64, 65, 1000, 8192, 8193, 8225, 20001])
def test_gradient_loss_and_logits(B):
    import torch

    from paper_2006_14952_amd import learned
    rng = np.random.default_rng(700 + B)
    X = (rng.standard_normal((B, 16)) * 2 + 1).astype(np.float32)
    y = rng.integers(0, 8, B).astype(np.int32)
    w = learned.init_params(3) + rng.standard_normal(5768).astype(np.float32) * np.float32(0.01)
    mu, isd = rng.standard_normal(16).astype(np.float32), (0.5 + rng.random(16)).astype(np.float32)
    cw = (0.5 + rng.random(8)).astype(np.float32)
    t = [torch.tensor(a, device="cuda") for a in (w, mu, isd, X, y, cw)]
    Z = learned.forward(t[0], t[1], t[2], t[3]).cpu().numpy()
    loss, g = learned.grad(*t)
    Z64 = omlp.forward(w, X, mu, isd)[3]
    l64, g64 = omlp.loss_and_grad(w, X, y, cw, mu, isd)
    # FP32 roundings: three layers of at most 64 terms, the weights' sum and the gradients' sums over the batch
    eps = 2.0 ** -24
    assert np.abs(Z - Z64).max() <= 3 * 64 * eps * np.abs(Z64).max()
    tol = eps * (200 + B)
    assert abs(loss - l64) <= tol * abs(l64)
    assert np.linalg.norm(g.cpu().numpy() - g64) <= tol * np.linalg.norm(g64)
    if B <= 8192:
        gn, ln = torch.full_like(g, np.nan), torch.full((1,), np.nan, device="cuda")
        learned.grad_noalloc(*t, gn, ln)
        assert abs(float(ln) - l64) <= eps * 400 * abs(l64)
        assert np.linalg.norm(gn.cpu().numpy() - g64) <= eps * 400 * np.linalg.norm(g64)
