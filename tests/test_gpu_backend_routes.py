"""Back-end routes that only larger calls take: whitening on the matrix cores
(more than 192 dimensions or 1024 rows) at sizes that are no whole tiles, and
trial scores through the matrix of all pairs (98,304 trials and more).

Sums are FP64 of FP32 inputs and round once to FP32: lnorm within 1e-6, scores
within 2e-6 (1 + |s| + sum of the absolute terms).
"""
import numpy as np
import pytest

from _gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dim", [(1025, 2), (1025, 33), (1040, 64), (17, 193), (15, 401), (1, 511)])
def test_whitened_length_norm_on_the_matrix_cores(n, dim):
    from paper_1906_08556_amd import ivx
    rng = np.random.default_rng(dim)
    X = rng.standard_normal((n, dim)).astype(np.float32)
    mean, W = rng.standard_normal(dim), rng.standard_normal((dim, dim))
    be = ivx.Backend(dim, n, 2)
    for m in (mean, None):
        y = (X.astype(np.float64) - (0 if m is None else m)) @ W.T
        y /= np.linalg.norm(y, axis=1, keepdims=True)
        got = be.lnorm(dev(X), None if m is None else dev(m), dev(W)).cpu().numpy()
        assert np.abs(got - y).max() <= 1e-6


@pytest.mark.parametrize("n1,n2,d,same", [(321, 315, 17, False), (321, 315, 200, False),
                                          (64, 1600, 33, False), (330, 330, 2, True)])
def test_trial_scores_through_the_matrix_of_all_pairs(n1, n2, d, same):
    from paper_1906_08556_amd import ivx
    rng = np.random.default_rng(n1 + d)
    Y1 = rng.standard_normal((n1, d)).astype(np.float32)
    Y2 = Y1 if same else rng.standard_normal((n2, d)).astype(np.float32)
    mu, A = 0.1 * rng.standard_normal(d), rng.standard_normal((d, d)) / np.sqrt(d)
    psi = rng.gamma(2, 1, d)
    be = ivx.Backend(max(2, d), max(n1, n2), 2)
    model = (dev(mu), dev(A), dev(psi))
    i, j = np.meshgrid(np.arange(n1), np.arange(n2), indexing="ij")
    allp = np.stack([i.ravel(), j.ravel()], 1).astype(np.int32)
    allp = allp[rng.permutation(len(allp))]
    assert len(allp) >= 98304
    z1, z2 = (Y1 - mu) @ A, (Y2 - mu) @ A
    det = (psi + 1) ** 2 - psi ** 2
    a, b = -0.5 * ((psi + 1) / det - 1 / (psi + 1)), psi / det
    c = (-0.5 * np.log(det) + np.log(psi + 1)).sum()
    ref = c + (a * z1 ** 2).sum(1)[:, None] + (a * z2 ** 2).sum(1)[None] + (b * z1) @ z2.T
    mag = (np.abs(a) * z1 ** 2).sum(1)[:, None] + (np.abs(a) * z2 ** 2).sum(1)[None] + \
        np.abs(b * z1) @ np.abs(z2).T
    k = (allp[:, 0], allp[:, 1])
    tol = (2e-6 * (1 + np.abs(ref) + mag))[k]
    d1 = dev(Y1)
    d2 = d1 if same else dev(Y2)
    s = be.plda_score(model, d1, d2, dev(allp)).cpu().numpy()
    assert np.all(np.abs(s - ref[k]) <= tol)
    be.status()
    bad = allp.copy()
    bad[0], bad[1], bad[2], bad[3] = (n1, 0), (-1, 0), (0, n2), (0, -1)
    s = be.plda_score(model, d1, d2, dev(bad)).cpu().numpy()
    assert np.isnan(s[:4]).all() and np.all(np.abs(s - ref[k])[4:] <= tol[4:])
    with pytest.raises(ivx.IvxError):
        be.status()
