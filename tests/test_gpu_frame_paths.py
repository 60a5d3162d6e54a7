"""Routes of the frame stage at the sizes where they can go wrong: block and
chunk edges of the component sort and of the exact scores.

Posteriors are scored in FP64 on both sides and rounded once to FP32, so an
entry is within 1e-6 of the oracle's and the frame log-likelihood within 1e-8;
n and f follow from the posteriors with a rounding of 2^-33 per term; S is an
FP64 sum of FP32-rounded posteriors (2e-7 of the absolute terms).
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from _gpu_helpers import dev, make_ctx, packed_upper

pytestmark = pytest.mark.gpu


def _lists(ctx, X, prec=0):
    F = X.shape[0]
    pi = torch.full((F, 16), -7, dtype=torch.int32, device="cuda")
    pv = torch.full((F, 16), -7.0, device="cuda")
    ll = torch.full((F,), -7.0, dtype=torch.float64, device="cuda")
    ctx.ubm_posteriors(X, post_idx=pi, post_val=pv, frame_ll=ll, prec=prec)
    ctx.sync_status()
    return pi.cpu().numpy(), pv.cpu().numpy(), ll.cpu().numpy()


def _dense(pi, pv, C):
    g = np.zeros((len(pi), C))
    t, s = np.nonzero(pi >= 0)
    g[t, pi[t, s]] = pv[t, s]
    return g


@pytest.mark.parametrize("C,F", [(1, 1), (63, 255), (65, 256), (65, 257), (130, 4095)])
def test_posteriors_and_statistics_at_block_edges(C, F):
    """One frame, one component, 64-component and 256-frame edges of the sort."""
    wl = synth.make(1, C=C, D=20, R=8, U=4, lengths=f"uniform:{F}:{F}", n_utts=1)
    ctx = make_ctx(wl)
    X, off = dev(wl.X), dev(wl.utt_off)
    pi, pv, ll = _lists(ctx, X)
    g_ref, lse = oracle.posteriors(oracle.frame_loglik(wl.X, wl.w, wl.mu, wl.cov))
    assert np.abs(_dense(pi, pv, C) - g_ref).max() <= 1e-6
    assert np.abs(ll - lse).max() <= 1e-8
    n = torch.empty(1, C, device="cuda")
    f = torch.empty(1, C, 20, device="cuda")
    S = torch.zeros(C, 210, dtype=torch.float64, device="cuda")
    ctx.bw_stats(X, off, n, f, S_acc=S)
    ctx.sync_status()
    n_ref, f_ref, S_ref = oracle.bw_stats(wl.X, wl.utt_off, g_ref)
    tol = 1e-6 * F * np.abs(wl.X).max()
    assert np.abs(n.cpu().numpy() - n_ref).max() <= 1e-6 * F
    assert np.abs(f.cpu().numpy() - f_ref).max() <= tol
    absS = np.einsum("tc,ti,tj->cij", g_ref, np.abs(wl.X), np.abs(wl.X))
    err = np.abs(S.cpu().numpy() - packed_upper(S_ref))
    assert np.all(err <= 2e-7 * packed_upper(absS) + 1e-9 + 1e-6 * np.abs(wl.X).max() ** 2)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("C,D", [(512, 32), (701, 62), (2048, 60)])
def test_bound_route_equals_dense_route(C, D, prec):
    """Large batches preselect components by a bound; the posterior lists are
    those of the dense kernel, bit for bit, on ordinary frames, on frames with
    many near-equal components (more than a list holds; far from
    the other frames, whose lists they would fill at the edge of the margin), and on frames that
    the bound cannot serve (features beyond FP16 scaling, not finite)."""
    from paper_1906_08556_amd import ivx
    F = 20011
    wl = synth.make(2, C=C, D=D, R=4, U=20, lengths="uniform:1001:1001")
    X = wl.X[:F].copy()
    mu, cov = wl.mu.copy(), wl.cov.copy()
    # the last 100 components nearly the same: frames drawn at their mean meet
    # lists of more than 32 candidates per half (last, so that the dense kernel
    # has the other components' scores before it counts candidates)
    mu[-100:] = mu[-1] + 50.0 + 1e-3 * np.arange(100)[:, None]
    cov[-100:] = cov[-1]
    rng = np.random.default_rng(5)
    X[100:140] = mu[-50] + rng.standard_normal((40, D)) @ np.linalg.cholesky(cov[-1]).T
    X[200:210] *= 1e4
    X[300] = 3e7      # beyond 2^23: the dense kernel's
    X[301, D - 1] = np.inf
    X[F - 1, 0] = np.nan
    ctx = ivx.Context(C, D, 4, 1, F)
    ctx.set_ubm(dev(wl.w), dev(mu), dev(cov))
    got = []
    for ncb in (8, 4):  # 8: the bound; an explicitly chosen shape: dense
        ctx.tuning_set(frame_ncb=ncb, frame_ncb_bf16=ncb)
        pi = torch.full((F, 16), -7, dtype=torch.int32, device="cuda")
        pv = torch.full((F, 16), -7.0, device="cuda")
        ll = torch.full((F,), -7.0, dtype=torch.float64, device="cuda")
        ctx.ubm_posteriors(dev(X), post_idx=pi, post_val=pv, frame_ll=ll, prec=prec)
        with pytest.raises(ivx.IvxError):  # the non-finite frames, the flat ones
            ctx.sync_status()
        got.append((pi.cpu().numpy(), pv.cpu().numpy(), ll.cpu().numpy()))
    assert np.all(got[0][0][100:140] >= C - 100)  # 16 of the near-equal ones
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("C,D,F", [(1, 3, 1), (63, 20, 15), (65, 20, 17), (130, 61, 33),
                                   (2048, 60, 1), (2048, 60, 100), (700, 63, 1030)])
def test_small_batch_route_equals_dense_route(C, D, F, prec):
    """Small batches split the scores over components: the same lists, bit for
    bit, as the dense kernel with 128 components per launch (component counts
    up to one launch, or far more, with well separated scores)."""
    wl = synth.make(2, C=C, D=D, R=4, U=1, lengths=f"uniform:{F}:{F}")
    ctx = make_ctx(wl)
    X = dev(wl.X)
    a = _lists(ctx, X, prec)
    ctx.tuning_set(frame_ncb=4, frame_ncb_bf16=4)
    b = _lists(ctx, X, prec)
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("C,D,F,k", [(1, 1, 1, 1), (64, 20, 33, 21), (40, 5, 127, 8),
                                     (130, 33, 129, 9), (257, 63, 130, 20), (300, 60, 257, 32)])
def test_pruned_alignment_at_list_and_tile_edges(C, D, F, k):
    """Frame log-likelihoods over the k best components of the diagonal UBM:
    FP64 of the kept proposals, so 1e-6 as for the larger workloads, wherever
    the k-th and the next diagonal score differ by more than the FP32 sums may
    (2 x 128 roundings of the terms' magnitude on either side)."""
    from paper_1906_08556_amd import ivx
    wl = synth.make(2, C=C, D=D, R=4, U=1, lengths=f"uniform:{F}:{F}")
    ctx = make_ctx(wl)
    ctx.pruned_set(k, 0.025)
    ll = torch.empty(F, dtype=torch.float64, device="cuda")
    ctx.ubm_posteriors(dev(wl.X), frame_ll=ll, sel=ivx.IVX_SEL_PRUNED)
    ctx.sync_status()
    lld = oracle.diag_frame_loglik(wl.X, wl.w, wl.mu, wl.cov)
    order = oracle.preselect(lld, min(k + 1, C))
    _, lse = oracle.pruned_posteriors(wl.X, wl.w, wl.mu, wl.cov, order[:, :k], 0.025)
    clear = np.ones(F, bool)
    if k < C:
        var = np.stack([np.diag(c) for c in wl.cov])
        x = np.abs(wl.X.astype(np.float64) - (wl.w[:, None] * wl.mu).sum(0))
        m = np.abs(wl.mu - (wl.w[:, None] * wl.mu).sum(0))
        mag = x @ (m / var).T + (x ** 2) @ (0.5 / var).T + (0.5 * m ** 2 / var).sum(1) + 4 * D
        gap = np.take_along_axis(lld, order[:, k - 1:k], 1) - np.take_along_axis(lld, order[:, k:], 1)
        clear = gap[:, 0] > 2 * 2 * 128 * 2.0 ** -24 * mag.max(1)
    assert clear.mean() > 0.5
    assert np.abs(ll.cpu().numpy() - lse)[clear].max() <= 1e-6


def test_bound_route_in_several_parts_equals_calls_of_one_part():
    """More frames than the sweeps keep sums for (131072 at C = 8192) against
    calls that fit: the same lists, bit for bit.  (Not the dense kernel: with
    8192 components its running list overflows in mid sweep for some frames,
    which then get their 16 best components instead of those in the margin.)"""
    C, D, F = 8192, 32, 131072 + 300
    wl = synth.make(2, C=C, D=D, R=4, U=2, lengths="uniform:1000:1000")
    rng = np.random.default_rng(8)
    X = wl.X[rng.integers(0, wl.F, F)] + 0.1 * rng.standard_normal((F, D)).astype(np.float32)
    ctx = make_ctx(wl, max_frames=F)
    a = _lists(ctx, dev(X))
    b = [_lists(ctx, dev(X[i:i + 40000])) for i in range(0, F, 40000)]
    for k in range(3):
        np.testing.assert_array_equal(a[k], np.concatenate([q[k] for q in b]))
