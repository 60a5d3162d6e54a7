"""The 128 x 128 tiles of the FP32 products (taken where the padded output is no
larger than with 64 x 64 tiles and 512 of them fill the device) at ragged edges:
the E-step's precision product and the selector's products.  Bounds as for these
steps elsewhere."""
import gc

import numpy as np
import pytest
import torch

import oracle
import synth
from _gpu_helpers import dev, make_ctx, unpack_upper

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,U", [(70, 120), (72, 500), (72, 1001)])  # 72: aligned rows of n
def test_estep_on_large_tiles(C, U):
    """i-vector cosine >= 0.9999, relative error and Phi relative Frobenius <= 2e-3."""
    R, D = 400, 20
    wl = synth.make(1, C=C, D=D, R=R, U=1)
    rng = np.random.default_rng(U)
    n = rng.gamma(2.0, 2.0, size=(U, C)).astype(np.float32)
    f = (n[:, :, None] * (wl.mu + rng.standard_normal((U, C, D)))).astype(np.float32)
    tv = oracle.init_tv(wl.mu, wl.cov, wl.T_init)
    ctx = make_ctx(wl, max_utts=U)
    ctx.set_tv(*(dev(a) for a in tv))
    phi = torch.empty(U, R, device="cuda")
    Phi = torch.empty(U, R * (R + 1) // 2, device="cuda")
    ctx.tv_estep(dev(n), dev(f), phi, Phi=Phi)
    ctx.sync_status()
    u = np.unique(np.r_[0:3, 62:66, 124:130, U // 2, U - 6:U])  # at tile edges and between
    u = u[u < U]
    e = oracle.estep(n[u].astype(np.float64), f[u].astype(np.float64), *tv)
    p = phi.cpu().numpy()[u]
    cos = (p * e["phi"]).sum(1) / np.linalg.norm(p, axis=1) / np.linalg.norm(e["phi"], axis=1)
    assert cos.min() >= 0.9999
    assert np.max(np.abs(p - e["phi"]) / np.abs(e["phi"]).max(1, keepdims=True)) <= 2e-3
    P = unpack_upper(Phi.cpu().numpy()[u], R)
    err = np.linalg.norm(P - e["Phi"], axis=(1, 2)) / np.linalg.norm(e["Phi"], axis=(1, 2))
    assert err.max() <= 2e-3


def test_selector_gradients_on_large_tiles():
    """Forward and weight-gradient products with 8188 rows and 2044 components; frames
    whose pre-activations lie within 1e-3 of zero are left out (FP32 rounding may
    choose the other ReLU branch).  Error below 1e-5 of the sum of the absolute
    terms, as at the smaller batch."""
    from paper_1906_08556_amd import ivx
    C, D, h1, h2, B = 2044, 20, 128, 512, 8188
    rng = np.random.default_rng(0)
    X = (2.0 * rng.standard_normal((24000, D))).astype(np.float32)
    params = synth.mlp_init(D, h1, h2, C, seed=2)
    mean, std = [a.astype(np.float32) for a in oracle.feature_stats(X)]
    pw = [p.astype(np.float64) for p in synth.mlp_split(params, D, h1, h2, C)]
    Xh = oracle.standardise(X, mean.astype(np.float64), std.astype(np.float64))
    a1 = Xh @ pw[0].T + pw[1]
    a2 = np.maximum(a1, 0) @ pw[2].T + pw[3]
    fidx = np.flatnonzero((np.abs(a1).min(1) > 1e-3) & (np.abs(a2).min(1) > 1e-3))[:B]
    assert len(fidx) == B
    ctx = ivx.Context(C, D, 2, 1, len(X))
    ctx.selector_set(dev(params), dev(mean), dev(std), H1=h1, H2=h2, k=20, max_train_batch=B)
    idx = np.full((len(X), 16), -1, np.int32)
    val = np.zeros((len(X), 16), np.float32)
    idx[:, 0] = rng.integers(0, C - 1, len(X))
    idx[:, 1] = idx[:, 0] + 1
    val[:, 0] = 0.5 + 0.5 * rng.random(len(X))
    val[:, 1] = 1.0 - val[:, 0]
    grad = torch.empty(ctx.selector_param_count(), dtype=torch.float32, device="cuda")
    ctx.selector_grad(dev(X), dev(fidx), dev(idx), dev(val), grad=grad)
    ctx.sync_status()
    gam = np.zeros((B, C))
    gam[np.arange(B), idx[fidx, 0]] = val[fidx, 0]
    gam[np.arange(B), idx[fidx, 1]] = val[fidx, 1]
    z, cache = oracle.mlp_forward(pw, Xh[fidx])
    ref = oracle.mlp_backward(pw, cache, z, gam)
    dz = (oracle.softmax(z) + gam) / B  # every quantity by its absolute value
    W2, W3 = np.abs(pw[2]), np.abs(pw[4])
    da2 = (dz @ W3) * (cache[3] > 0)
    da1 = (da2 @ W2) * (cache[1] > 0)
    mag = (da1.T @ np.abs(cache[0]), da1.sum(0), da2.T @ np.abs(cache[2]), da2.sum(0),
           dz.T @ np.abs(cache[4]), dz.sum(0))
    for g, r, m in zip(synth.mlp_split(grad.cpu().numpy(), D, h1, h2, C), ref, mag):
        assert np.linalg.norm(g - r) <= 1e-5 * np.linalg.norm(m)


def test_memory_of_a_wide_selector():
    """Hidden layers of 4096: the partial products of the split weight gradients take
    at most 64 MB beside the training batch's own arrays (16 frames here, the column
    sums' 32 rows, 8 MB for allocation granules)."""
    from paper_1906_08556_amd import ivx
    C, D, H, B = 300, 20, 4096, 16
    rng = np.random.default_rng(1)
    params = dev((0.01 * rng.standard_normal(H * (D + 1) + H * (H + 1) + C * (H + 1))).astype(np.float32))
    mean, std = dev(np.zeros(D, np.float32)), dev(np.ones(D, np.float32))
    ctx = ivx.Context(C, D, 2, 1, 64)

    def free(batch):
        ctx.selector_set(params, mean, std, H1=H, H2=H, k=20, max_train_batch=batch)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    gc.collect()  # contexts of other tests
    free(0)
    a = free(0)
    assert a - free(B) <= (64 << 20) + 4 * (B * 8 * H + 32 * H) + (8 << 20)
