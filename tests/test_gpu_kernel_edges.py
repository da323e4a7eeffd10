"""Kernels at the edges of their tiles and dispatch rules (remainders, the
smallest and largest sizes of a range), against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()
    from paper_2010_10131_amd import api as a
    return a


@pytest.mark.parametrize("B", [31, 32, 33, 64, 4499])
def test_mlp_gradient_at_workgroup_edges(api, B):
    """32 samples per workgroup: one workgroup writes the gradient itself,
    several write partial sums.  FP32 products and sums of 32 samples, FP64
    above: within 2^-24 times a few hundred operations of the oracle, relative
    to the largest entry."""
    import torch
    from test_gpu_selector import rand_params, unpack
    p = rand_params(B)
    rng = np.random.default_rng(B)
    X = rng.standard_normal((10, B)).astype(np.float32)
    T = rng.standard_normal((2, B)).astype(np.float32)
    dev = [torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t() for a in (X, T)]
    loss, grad = api.mlp_loss_grad(torch.from_numpy(p).cuda(), *dev)
    Ws, bs, mu, isd = unpack(p.astype(np.float64))
    lo, dW, db = oracle.mlp_loss_grad(Ws, bs, (X.astype(np.float64) - mu[:, None]) * isd[:, None],
                                      T.astype(np.float64))
    go = np.concatenate([dW[0].T.ravel(), db[0], dW[1].T.ravel(), db[1], dW[2].T.ravel(), db[2], np.zeros(20)])
    assert abs(float(loss.item()) - lo) <= 1e-5 * lo
    np.testing.assert_allclose(grad.cpu().numpy(), go, rtol=0, atol=2e-5 * np.abs(go).max())
