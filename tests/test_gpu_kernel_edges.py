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


@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims,n,R", [((4, 8, 1), 1, 1), ((4, 3, 5), 1, 17), ((12, 32, 7), 1, 48), ((20, 33, 9), 1, 200),
                                      ((64, 64, 3), 1, 16), ((8, 65, 11), 1, 5), ((132, 97, 2), 1, 33),
                                      ((16, 300, 5), 1, 64), ((4, 20, 6), 2, 700), ((6, 40, 5), 1, 10)])
def test_strided_ttm_in_vectors(api, dims, n, R, prec):
    """Strided rows in 16-byte vectors (L a multiple of 4 values, or of 2 in
    FP64): last blocks that are not whole, contractions of one chunk, of two and
    beyond, r-tiles in one range and in several.  FP32 sums of K products (FP64
    ones: K eps), rounded to the data type."""
    dtype = "float64" if prec == "f64" else "float32"
    rng = np.random.default_rng(sum(dims) + R)
    Y = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    U = np.asfortranarray(rng.standard_normal((dims[n], R)))
    Z = api.to_numpy(api.ttm_mode_n(api.to_device(Y), api.to_device(U), n, "fp64" if prec == "f64" else prec))
    ref, bound = oracle.ttm_tensor(Y, U.T, n), oracle.ttm_tensor(np.abs(Y), np.abs(U).T, n)
    K = dims[n]
    unit = {"f64": 4 * K * 2.2e-16, "fp64": 2.0 ** -23, "fp32": (K + 2) * 2.0 ** -23,
            "bf16x3": (K + 2) * 2.0 ** -23 + 2.0 ** -15, "bf16x6": (K + 6) * 2.0 ** -23}[prec]
    assert np.all(np.abs(Z - ref) <= unit * bound + 1e-30)


@pytest.mark.parametrize("dims,ranks", [((20, 12, 9), (5, 6, 4)), ((8, 10, 37), (3, 5, 33)), ((36, 9, 50), (4, 3, 40))])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_error_sums_in_vectors(api, dims, ranks, dtype):
    """The fused error sums on tensors whose last mode has strided rows in whole
    vectors, against the oracle's reconstruction; the squares of differences of
    order one are summed in FP64."""
    rng = np.random.default_rng(sum(dims))
    G = np.asfortranarray(rng.standard_normal(ranks).astype(dtype))
    U = [np.asfortranarray(np.linalg.qr(rng.standard_normal((d, r)))[0]) for d, r in zip(dims, ranks)]
    X = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    out = api.tucker_error(api.to_device(X), api.to_device(G), [api.to_device(u) for u in U],
                           "fp64" if dtype == "float64" else "fp32").cpu().numpy()
    Xo = oracle.reconstruct(G.astype(np.float64), U)
    tol = 1e-12 if dtype == "float64" else 1e-5
    np.testing.assert_allclose(out, [np.sum((X - Xo) ** 2), np.sum(X.astype(np.float64) ** 2)], rtol=tol)


@pytest.mark.parametrize("R", [1, 2, 15, 16, 17, 32, 33, 64, 65, 80, 113, 127, 128])
def test_cholesky_qr_orders(api, R):
    """The blocked Cholesky and its inverse at the edges of its 16-column panels,
    through the ALS branch's QR of an I x R basis of an exactly rank-R unfolding.
    Two Cholesky-QR passes leave ||U^T U - I|| <= 6 (I R + R (R + 1)) u (Yamamoto
    et al., 2015); the basis spans the unfolding within the same bound."""
    I = 300
    rng = np.random.default_rng(R)
    Y = np.asfortranarray(rng.standard_normal((I, R)) @ rng.standard_normal((R, 3 * R)))
    Z, U, _, _ = api.mode_step(api.to_device(Y), 0, R, "als", "fp64", "fp64", seed=3)
    U = api.to_numpy(U)
    bound = 6 * (I * R + R * (R + 1)) * 1.1e-16
    assert np.linalg.norm(U.T @ U - np.eye(R), 2) <= bound
    assert np.linalg.norm(Y - U @ (U.T @ Y), 2) <= bound * np.linalg.norm(Y, 2)
    np.testing.assert_allclose(api.to_numpy(Z), U.T @ Y, rtol=0, atol=bound * np.linalg.norm(Y, 2))


@pytest.mark.parametrize("n,R", [(129, 1), (129, 110), (144, 8), (160, 32), (161, 33), (191, 60), (257, 64), (320, 112),
                                 (511, 17), (512, 80)])
def test_subspace_iteration_orders(api, n, R):
    """The subspace iteration's products, Cholesky-QR and finish at the edges of
    their tiles (16 rows and columns, 32-long contraction steps, odd and even
    orders), on a graded spectrum.  Accepted pairs have residuals within
    16 sqrt(n) eps ||S||, the Gram itself is within K eps of the one formed here;
    Cholesky-QR leaves ||U^T U - I|| <= 6 (n p + p (p + 1)) u with p <= 128."""
    rng = np.random.default_rng(n + R)
    K = n + 3
    sv = 0.93 ** np.arange(n)
    Y = np.asfortranarray((np.linalg.qr(rng.standard_normal((n, n)))[0] * sv)
                          @ np.linalg.qr(rng.standard_normal((K, n)))[0].T)
    S = Y @ Y.T
    _, U, ev, _ = api.mode_step(api.to_device(Y), 0, R, "eig", "fp64", "fp64")
    U, ev = api.to_numpy(U), ev.cpu().numpy()
    eps = 2.2e-16
    tol = (16 * np.sqrt(n) + 2 * K) * eps
    np.testing.assert_allclose(ev, sv[:R] ** 2, rtol=0, atol=tol)
    assert np.linalg.norm(S @ U - U * ev, axis=0).max() <= tol
    assert np.linalg.norm(U.T @ U - np.eye(R), 2) <= 6 * (n * 128 + 128 * 129) * eps / 2
    top = np.abs(U).argmax(0)
    assert np.all(U[top, np.arange(R)] > 0)


@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims,n", [((5, 3), 0), ((1, 700), 0), ((3, 65), 0), ((4, 33), 0), ((5, 1000), 0), ((33, 129), 0),
                                    ((96, 4100), 0), ((97, 515), 0), ((130, 301), 0), ((159, 2050), 0), ((160, 31), 0),
                                    ((161, 700), 0), ((163, 97), 0), ((256, 545), 0), ((258, 33), 0),
                                    ((7, 130, 5), 1), ((8, 33, 12), 1), ((9, 65, 40), 1), ((40, 129, 3), 1),
                                    ((31, 20, 17), 1), ((1, 200, 9), 1), ((24, 257), 1), ((36, 150, 40), 1),
                                    ((2, 65, 33), 1), ((6, 64, 64), 1)])
def test_gram_edges(api, dims, n, prec):
    """Grams at the edges of their tiles, stages and loaders: rows and columns
    beyond whole quads, octets across fibres, a last chunk that is not full.  FP32 accumulates 128 products at most
    (128 eps32 of the sum of magnitudes, doubled), bf16x3 drops products below
    2^-16, FP64 stays within K eps."""
    rng = np.random.default_rng(sum(dims) + n)
    X = np.asfortranarray(rng.standard_normal(dims).astype(np.float64 if prec == "f64" else np.float32))
    Xd = api.to_device(X)
    S = api.to_numpy(api.gram_mode_n(Xd, n, "fp64" if prec == "f64" else prec))
    M = np.moveaxis(X.astype(np.float64), n, 0).reshape(dims[n], -1)
    c = {"f64": 4 * M.shape[1] * 2.2e-16, "fp64": 4 * M.shape[1] * 2.2e-16, "fp32": 256 * 2.0 ** -24, "bf16x6": 256 * 2.0 ** -24,
         "bf16x3": 256 * 2.0 ** -24 + 4 * 2.0 ** -16}[prec]
    assert np.all(np.abs(S - M @ M.T) <= c * (np.abs(M) @ np.abs(M).T))
    np.testing.assert_array_equal(S, S.T)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("dims,n", [((1, 131073), 0), ((5, 140003), 0), ((20, 131072), 0), ((21, 140001), 0), ((40, 65537), 0),
                                    ((41, 33001), 0), ((80, 32769), 0), ((81, 33000), 0), ((4, 20, 32770), 1),
                                    ((36, 1, 3650), 1), ((28, 40, 2345), 1), ((8, 33, 8193), 1), ((12, 80, 2731), 1)])
def test_gram_of_short_rows(api, dims, n, dtype):
    """FP64 products of few rows over many columns: stages of 32 to 256 columns,
    rows that end within a stage, contiguous and strided.  K eps of the sums of
    magnitudes."""
    rng = np.random.default_rng(sum(dims))
    X = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    S = api.to_numpy(api.gram_mode_n(api.to_device(X), n, "fp64"))
    M = np.moveaxis(X.astype(np.float64), n, 0).reshape(dims[n], -1)
    assert np.all(np.abs(S - M @ M.T) <= 4 * M.shape[1] * 2.2e-16 * (np.abs(M) @ np.abs(M).T))
    np.testing.assert_array_equal(S, S.T)


def best_ms(call, reps=6, calls=10):
    """Time of a call: best of several runs of calls one after the other, by events
    on the stream, after one to warm up."""
    import torch
    call()
    times = []
    for _ in range(reps):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(calls):
            call()
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / calls)
    return min(times)


@pytest.mark.parametrize("I", [16, 24, 32])
def test_gram_of_short_rows_is_bound_by_its_reads(api, I):
    """An FP64 Gram of few rows has little to multiply: over 512 MB it takes no
    more than one and a half times a copy of the same data."""
    import torch
    X = torch.randn((2 ** 26 // I, I), dtype=torch.float64, device="cuda").t()
    to = torch.empty_like(X)
    gram, copy = best_ms(lambda: api.gram_mode_n(X, 0, "fp64")), best_ms(lambda: to.copy_(X))
    assert gram <= 1.5 * copy, (gram, copy)


@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims", [(95, 70, 5), (97, 20, 7), (100, 130, 9), (129, 65, 8), (201, 66, 1), (1001, 129, 2), (31, 161, 33)])
def test_gram_and_ttt_across_fibres(api, dims, prec):
    """Strided rows whose fibres are not whole octets: chunks within a fibre, across
    two and across several, and a last one that is not full.  Tolerances as in
    test_gram_edges."""
    rng = np.random.default_rng(sum(dims))
    dtype = np.float64 if prec == "f64" else np.float32
    X = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    Z = np.asfortranarray(rng.standard_normal((dims[0], 17, dims[2])).astype(dtype))
    p = "fp64" if prec == "f64" else prec
    M, N = (np.moveaxis(a.astype(np.float64), 1, 0).reshape(a.shape[1], -1) for a in (X, Z))
    c = {"f64": 4 * M.shape[1] * 2.2e-16, "fp64": 4 * M.shape[1] * 2.2e-16, "fp32": 256 * 2.0 ** -24, "bf16x6": 256 * 2.0 ** -24,
         "bf16x3": 256 * 2.0 ** -24 + 4 * 2.0 ** -16}[p if p != "f64" else "fp64"]
    S = api.to_numpy(api.gram_mode_n(api.to_device(X), 1, p))
    assert np.all(np.abs(S - M @ M.T) <= c * (np.abs(M) @ np.abs(M).T))
    P = api.to_numpy(api.ttt_mode_n(api.to_device(X), api.to_device(Z), 1, p))
    assert np.all(np.abs(P - M @ N.T) <= c * (np.abs(M) @ np.abs(N).T))


def test_gram_of_odd_fibres_keeps_up_with_whole_ones(api):
    """Long fibres that are not whole octets cost little more than whole ones: at
    most one and a half times (within a fibre every load is as wide)."""
    import torch
    def gram(L):
        X = torch.randn((60, 300, L), dtype=torch.float32, device="cuda").permute(2, 1, 0)
        return best_ms(lambda: api.gram_mode_n(X, 1, "bf16x3"))
    odd, whole = gram(1001), gram(1000)
    assert odd <= 1.5 * whole, (odd, whole)


def strided_ttm(api, dims, R, prec, seed):
    """One TTM along mode 1 against numpy: FP32 sums of K products (FP64 ones: K
    eps), rounded to the data type."""
    rng = np.random.default_rng(seed)
    dtype = np.float64 if prec == "f64" else np.float32
    K = dims[1]
    Y = np.asfortranarray(rng.standard_normal(dims).astype(dtype))
    U = np.asfortranarray(rng.standard_normal((K, R)))
    Z = api.to_numpy(api.ttm_mode_n(api.to_device(Y), api.to_device(U), 1, "fp64" if prec == "f64" else prec))
    Yf = Y.transpose(1, 0, 2).reshape(K, -1).astype(np.float64)
    ref, bound = U.T @ Yf, np.abs(U).T @ np.abs(Yf)
    unit = {"f64": 4 * K * 2.2e-16, "fp64": 2.0 ** -23, "fp32": (K + 2) * 2.0 ** -23,
            "bf16x3": (K + 2) * 2.0 ** -23 + 2.0 ** -15, "bf16x6": (K + 6) * 2.0 ** -23}[prec]
    assert np.all(np.abs(Z.transpose(1, 0, 2).reshape(R, -1) - ref) <= unit * bound + 1e-30)


@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims,R", [((44, 70, 7001), 64), ((44, 70, 7001), 10), ((1004, 66, 303), 33), ((262148, 97, 1), 17),
                                    ((44, 129, 2501), 60), ((36, 100, 1001), 40), ((36, 100, 1001), 7), ((36, 100, 1001), 100),
                                    ((20, 130, 121), 64), ((8, 200, 1251), 20), ((28, 80, 6001), 130)])
def test_strided_ttm_over_many_rows(api, dims, R, prec):
    """The streaming kernel where a wave goes from one block of rows to the next
    (the place in the tensor is carried along and wraps within the fibre), with a
    last block that is not full, and its forms of two, four and eight waves, beside
    the row counts where the general kernel takes over."""
    strided_ttm(api, dims, R, prec, sum(dims) + R)


def test_strided_ttm_reads_its_input_once(api):
    """512 x 64 over 131 K rows, one workgroup of eight waves short of filling the
    chip: at most four fifths of a copy of the 267 MB."""
    import torch
    Y = torch.randn((8160, 512, 16), dtype=torch.float32, device="cuda").permute(2, 1, 0)
    U = api.ttm_factor_prepare(torch.randn((64, 512), dtype=torch.float64, device="cuda").t(), "bf16x3")
    to = torch.empty_like(Y)
    ttm, copy = best_ms(lambda: api.ttm_mode_n_prepared(Y, U, 1, 64, "bf16x3")), best_ms(lambda: to.copy_(Y))
    assert ttm <= 0.8 * copy, (ttm, copy)


@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims,R", [((44, 40, 7001), 100), ((1004, 20, 303), 16), ((262148, 33, 1), 17), ((36, 64, 1001), 200),
                                    ((4, 50, 16), 700), ((100, 50, 50), 100), ((28, 7, 3001), 70), ((8, 32, 9), 1000)])
def test_expansion_over_many_rows_and_few(api, dims, R, prec):
    """The expansion kernel where a wave goes from one block of rows to the next,
    and where few rows are spread over ranges of r-tiles, down to one tile each."""
    strided_ttm(api, dims, R, prec, sum(dims) + R)


@pytest.mark.parametrize("dims,ranks", [((300, 1004, 37), (3, 4, 20)), ((44, 7001, 80), (4, 3, 40)), ((100, 100, 100), (5, 6, 50)),
                                        ((200, 152, 336), (4, 5, 40)), ((2, 2, 500), (2, 2, 4)), ((4, 2, 2100), (2, 2, 3))])
@pytest.mark.parametrize("prec", ["f64", "fp64", "fp32", "bf16x6"])
def test_error_sums_over_many_rows_and_few(api, dims, ranks, prec):
    """The fused error sums in the same forms: the partial sums of every workgroup
    and range are added up, each value once."""
    import torch
    dtype = torch.float64 if prec == "f64" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(sum(dims))
    def column_major(shape, t):
        return torch.randn(shape[::-1], generator=gen, device="cuda", dtype=t).permute(*range(len(shape) - 1, -1, -1))
    G, X = column_major(ranks, dtype), column_major(dims, dtype)
    U = [column_major((d, r), torch.float64) / d ** 0.5 for d, r in zip(dims, ranks)]
    U = [u.t().contiguous().t() for u in U]
    out = api.tucker_error(X, G, U, "fp64" if prec == "f64" else prec).cpu().numpy()
    T = G.double()
    for n, u in enumerate(U):   # G x_n U_n
        T = torch.tensordot(u, T, dims=([1], [n])).movedim(0, n)
    want = [float(((X.double() - T) ** 2).sum()), float((X.double() ** 2).sum())]
    np.testing.assert_allclose(out, want, rtol=1e-12 if prec == "f64" else 1e-5)


def test_small_expansion_spreads_over_the_chip(api):
    """50 -> 100 over 5000 rows has 80 blocks of rows: in one range of r-tiles most
    CUs had nothing to do.  Ten times the outputs in at most twice the time."""
    import torch
    Y = torch.randn((50, 50, 100), dtype=torch.float32, device="cuda").permute(2, 1, 0)
    def expand(R):
        U = api.ttm_factor_prepare(torch.randn((R, 50), dtype=torch.float64, device="cuda").t(), "fp32")
        Z = api.ttm_mode_n_prepared(Y, U, 1, R, "fp32")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                api.ttm_mode_n_prepared(Y, U, 1, R, "fp32", out=Z)
        return best_ms(g.replay, calls=2)
    many, few = expand(320), expand(32)
    assert many <= 2 * few, (many, few)


@pytest.mark.parametrize("K,R,L,M,dtype", [(1000, 5, 30, 1000, "float64"), (1000, 33, 30, 1000, "float64"), (1000, 33, 30, 1000, "float32"),
                                           (1000, 33, 1, 30000, "float64"), (1000, 33, 1, 30000, "float32")])
def test_long_contraction_over_many_rows(api, K, R, L, M, dtype):
    """30000 rows are enough for the general kernel, which has CUs to spare until
    then: at most 1.75 times the time of half the rows (the waves of a workgroup
    splitting K are bound by what they read and took twice the time)."""
    import torch
    t = getattr(torch, dtype)
    U = api.ttm_factor_prepare(torch.randn((R, K), dtype=torch.float64, device="cuda").t(), "fp64")
    def time(m):
        Y = torch.randn((m, K, L), dtype=t, device="cuda").permute(2, 1, 0)
        Y, n = (Y, 1) if L > 1 else (Y.reshape(K, m), 0)
        Z = api.ttm_mode_n_prepared(Y, U, n, R, "fp64")
        return best_ms(lambda: api.ttm_mode_n_prepared(Y, U, n, R, "fp64", out=Z))
    whole, half = time(M), time(M // 2)
    assert whole <= 1.75 * half, (whole, half)


@pytest.mark.parametrize("levels", [(1.0, 1e-12), (1.0, 1e-4), (1.0, 0.5, 0.25)])
@pytest.mark.parametrize("n", [16, 33, 64, 100, 128])
def test_direct_solver_on_large_clusters(api, n, levels):
    """Two or three eigenvalues that many eigenvectors share: Gram-Schmidt inside a
    cluster must not magnify what a vector has outside its eigenspace.  The solver's
    shifts lie within 32 eps ||T|| of the eigenvalues, ||T|| <= 2 ||S||: residuals
    within 64 n eps ||S||."""
    for seed in range(3):
        rng = np.random.default_rng(n + seed)
        Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
        Y = np.asfortranarray(Q * np.sqrt(np.array(levels)[(len(levels) * np.arange(n)) // n]))
        S = Y @ Y.T
        for R in ((n + 1) // 2, n):
            _, U, ev, _ = api.mode_step(api.to_device(Y), 0, R, "eig", "fp64", "fp64")
            U, ev = api.to_numpy(U), ev.cpu().numpy()
            assert np.linalg.norm(S @ U - U * ev, 2) <= 64 * n * 2.2e-16
            np.testing.assert_allclose(U.T @ U, np.eye(R), rtol=0, atol=8 * n * 2.2e-16)
