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


@pytest.mark.parametrize("spectrum", ["graded", "clustered"])
@pytest.mark.parametrize("n,R", [(1, 1), (2, 2), (3, 2), (4, 4), (17, 16), (18, 17), (49, 8), (63, 63), (64, 64),
                                 (65, 64), (65, 65), (80, 64), (81, 33), (96, 96), (113, 65), (127, 127),
                                 (128, 1), (128, 100), (128, 128)])
def test_direct_solver_orders(api, n, R, spectrum):
    """The direct solver of the decompositions at the edges of its register
    layout (64 rows a wave, 16-column tiles, 16-reflector blocks, blocks that do
    or do not fit the LDS): a 2-way FP64 tensor whose mode-1 Gram has known
    eigenvalues, some of them equal.  Residual and orthogonality of a
    backward-stable solver: a few n eps ||S||, here within 8 n eps."""
    rng = np.random.default_rng(n * 131 + R)
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    sv = 0.9 ** np.arange(n) if spectrum == "graded" else 1.0 / (1.0 + np.arange(n) // 3)
    Y = np.asfortranarray(Q * sv)
    S = Y @ Y.T
    _, U, ev, _ = api.mode_step(api.to_device(Y), 0, R, "eig", "fp64", "fp64")
    U, ev = api.to_numpy(U), ev.cpu().numpy()
    tol = 8 * n * 2.2e-16
    np.testing.assert_allclose(ev, np.sort(sv ** 2)[::-1][:R], rtol=0, atol=max(tol, 1e-15))
    assert np.linalg.norm(S @ U - U * ev, 2) <= max(tol, 1e-15)
    np.testing.assert_allclose(U.T @ U, np.eye(R), rtol=0, atol=max(tol, 1e-15))
    top = np.abs(U).argmax(0)
    assert np.all(U[top, np.arange(R)] > 0)


def within(Z, ref, bound, K):
    """FP64 products and sums of K terms: K eps of the sum of magnitudes."""
    assert np.all(np.abs(Z - ref) <= 4 * K * 2.2e-16 * bound + 1e-300)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("dims,R", [((65, 40), 1), ((67, 2001), 16), ((130, 700), 17), ((4097, 33), 33),
                                    ((601, 1), 64), ((9000, 300), 10), ((96, 20, 9), 20)])
def test_narrow_ttt(api, dims, R, dtype):
    """TTT over the first mode with few columns of the second operand: odd row
    counts, one to four column tiles, one and several column ranges."""
    rng = np.random.default_rng(sum(dims) + R)
    Y = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    Z = np.asfortranarray(rng.standard_normal((R,) + dims[1:]).astype(dtype))
    P = api.to_numpy(api.ttt_mode_n(api.to_device(Y), api.to_device(Z), 0, "fp64"))
    Yn, Zn = oracle.unfold(Y, 0), oracle.unfold(Z, 0)
    within(P, oracle.ttt(Yn, Zn), oracle.ttt(np.abs(Yn), np.abs(Zn)), Yn.shape[1])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("dims,n,R", [((993, 40), 0, 5), ((1025, 17), 0, 33), ((1024, 1), 0, 16), ((7, 1100, 3), 1, 20),
                                      ((30, 2000), 1, 50), ((5000, 2, 3), 0, 70)])
def test_long_contraction_ttm(api, dims, n, R, dtype):
    """FP64-product TTM with a long mode and few rows (eight waves split the
    contraction): ragged chunks, rows and r-tiles, contiguous and strided rows."""
    rng = np.random.default_rng(sum(dims) + R)
    Y = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    U = np.asfortranarray(rng.standard_normal((dims[n], R)))
    Z = api.to_numpy(api.ttm_mode_n(api.to_device(Y), api.to_device(U), n, "fp64"))
    ref, bound = oracle.ttm_tensor(Y, U.T, n), oracle.ttm_tensor(np.abs(Y), np.abs(U).T, n)
    if dtype == "float32":
        assert np.all(np.abs(Z - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-9 * bound)
    else:
        within(Z, ref, bound, dims[n])
