"""Routes of the E-step by the number of utterances: rows of A on the vector
units (up to 16 utterances), 64 x 64 and 128 x 128 MFMA tiles, with and without
the covariance.  Bounds as for the E-step elsewhere: i-vector cosine >= 0.9999,
relative error <= 2e-3, Phi relative Frobenius <= 2e-3."""
import numpy as np
import pytest
import torch

import oracle
import synth
from _gpu_helpers import dev, make_ctx, unpack_upper

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [45, 160])
@pytest.mark.parametrize("U", [1, 2, 3, 8, 9, 16, 17, 64, 65, 129])
def test_estep_by_number_of_utterances(U, R):
    wl = synth.make(1, C=70, D=20, R=R, U=1)
    rng = np.random.default_rng(U)
    n = rng.gamma(2.0, 2.0, size=(U, 70)).astype(np.float32)
    f = (n[:, :, None] * (wl.mu + rng.standard_normal((U, 70, 20)))).astype(np.float32)
    tv = oracle.init_tv(wl.mu, wl.cov, wl.T_init)
    ctx = make_ctx(wl, max_utts=U)
    ctx.set_tv(*(dev(a) for a in tv))
    e = oracle.estep(n.astype(np.float64), f.astype(np.float64), *tv)
    phi = torch.empty(U, R, device="cuda")
    Phi = torch.empty(U, R * (R + 1) // 2, device="cuda")
    ctx.tv_estep(dev(n), dev(f), phi, Phi=Phi)
    only = torch.empty(U, R, device="cuda")
    ctx.tv_estep(dev(n), dev(f), only)
    ctx.sync_status()
    p = phi.cpu().numpy()
    cos = (p * e["phi"]).sum(1) / np.linalg.norm(p, axis=1) / np.linalg.norm(e["phi"], axis=1)
    assert cos.min() >= 0.9999
    assert np.max(np.abs(p - e["phi"]) / np.abs(e["phi"]).max(1, keepdims=True)) <= 2e-3
    P = unpack_upper(Phi.cpu().numpy(), R)
    err = np.linalg.norm(P - e["Phi"], axis=(1, 2)) / np.linalg.norm(e["Phi"], axis=(1, 2))
    assert err.max() <= 2e-3
    np.testing.assert_array_equal(only.cpu().numpy(), p)
