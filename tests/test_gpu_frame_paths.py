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
