"""Routes of the scoring back-end at their edges: whitened length norm at tile
remainders, PLDA trials one by one and through the matrix of all pairs.

Sums are FP64 of FP32 inputs and round once to FP32: lnorm within 1e-6, scores
within 2e-6 (1 + |s| + sum of the absolute terms), as FP32 storage of the
projected vectors (6e-8 relative each) allows.
"""
import numpy as np
import pytest

from _gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dim", [(1, 2), (15, 16), (17, 33), (64, 100), (33, 512)])
def test_lnorm_with_and_without_whitening(n, dim):
    from paper_1906_08556_amd import ivx
    rng = np.random.default_rng(dim)
    X = rng.standard_normal((n, dim)).astype(np.float32)
    mean, W = rng.standard_normal(dim), rng.standard_normal((dim, dim))
    be = ivx.Backend(max(2, dim), n, 2)
    for m, w in ((mean, W), (None, W), (mean, None), (None, None)):
        y = X.astype(np.float64) - (0 if m is None else m)
        if w is not None:
            y = y @ w.T
        y /= np.linalg.norm(y, axis=1, keepdims=True)
        got = be.lnorm(dev(X), None if m is None else dev(m), None if w is None else dev(w))
        assert np.abs(got.cpu().numpy() - y).max() <= 1e-6


@pytest.mark.parametrize("dim", [2, 3, 31, 512])
def test_eigendecomposition_at_smallest_odd_and_largest_order(dim):
    from paper_1906_08556_amd import ivx
    rng = np.random.default_rng(dim)
    n = 4 * dim + 10
    X = (rng.standard_normal((n, dim)) * rng.uniform(0.5, 2.0, dim)).astype(np.float32)
    mean, W = ivx.Backend(dim, n, 2).whitening(dev(X))
    W = W.cpu().numpy()
    cov = np.cov(X.astype(np.float64).T, bias=True)
    # off-diagonal norm 1e-13 of the whole, condition below 1e3: 1e-9 leaves a factor of ten
    assert np.abs(W @ cov @ W.T - np.eye(dim)).max() <= 1e-9
    np.testing.assert_allclose(mean.cpu().numpy(), X.astype(np.float64).mean(0), atol=1e-12)


@pytest.mark.parametrize("n1,n2,d", [(1, 1, 2), (65, 64, 17), (130, 63, 200)])
def test_plda_scores_one_by_one_and_by_matrix(n1, n2, d):
    from paper_1906_08556_amd import ivx
    rng = np.random.default_rng(n1)
    Y1 = rng.standard_normal((n1, d)).astype(np.float32)
    Y2 = rng.standard_normal((n2, d)).astype(np.float32)
    mu, A = 0.1 * rng.standard_normal(d), rng.standard_normal((d, d)) / np.sqrt(d)
    psi = rng.gamma(2, 1, d)
    be = ivx.Backend(max(2, d), max(n1, n2), 2)
    model = (dev(mu), dev(A), dev(psi))
    i, j = np.meshgrid(np.arange(n1), np.arange(n2), indexing="ij")
    allp = np.stack([i.ravel(), j.ravel()], 1).astype(np.int32)
    z1, z2 = (Y1 - mu) @ A, (Y2 - mu) @ A
    det = (psi + 1) ** 2 - psi ** 2
    a, b = -0.5 * ((psi + 1) / det - 1 / (psi + 1)), psi / det
    c = (-0.5 * np.log(det) + np.log(psi + 1)).sum()
    ref = c + (a * z1 ** 2).sum(1)[:, None] + (a * z2 ** 2).sum(1)[None] + (b * z1) @ z2.T
    mag = (np.abs(a) * z1 ** 2).sum(1)[:, None] + (np.abs(a) * z2 ** 2).sum(1)[None] + \
        np.abs(b * z1) @ np.abs(z2).T
    tol = 2e-6 * (1 + np.abs(ref) + mag)
    full = be.plda_score(model, dev(Y1), dev(Y2), dev(allp)).cpu().numpy().reshape(n1, n2)
    assert np.all(np.abs(full - ref) <= tol)
    few = allp[:max(1, n1 * n2 // 20)]  # too few for the matrix
    one = be.plda_score(model, dev(Y1), dev(Y2), dev(few)).cpu().numpy()
    k = (few[:, 0], few[:, 1])
    assert np.all(np.abs(one - ref[k]) <= tol[k])
    be.status()
    bad = allp.copy()
    bad[0] = (n1, 0)
    s = be.plda_score(model, dev(Y1), dev(Y2), dev(bad)).cpu().numpy()
    assert np.isnan(s[0]) and np.isfinite(s[1:]).all()
    with pytest.raises(ivx.IvxError):
        be.status()
