"""ubm_posteriors_static with batches beyond the context's own size, and beside
calls of the same context on another stream.

Both entry points take their candidate lists from the same scores and rescore
them with the same FP64 arithmetic, so lists and values are the same bits.
"""
import numpy as np
import pytest
import torch

import synth
from _gpu_helpers import dev, make_ctx

pytestmark = pytest.mark.gpu


def _lists(F):
    return (torch.full((F, 16), -7, dtype=torch.int32, device="cuda"),
            torch.full((F, 16), -7.0, device="cuda"),
            torch.full((F,), -7.0, dtype=torch.float64, device="cuda"))


def _ms(call):
    call()
    t = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b))
    return min(t)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("F", [8300, 20000, 140000])  # 140,000: two frame blocks per wave
def test_static_call_of_a_small_context(F, prec):
    """The batch is bounded by the library's array, not by the context; the call
    takes about as long as that of a context made for the batch (a factor of 4
    leaves room for the second sweep's extra products)."""
    wl = synth.make(2, R=4, U=20, lengths="uniform:1000:1000")
    rng = np.random.default_rng(F)
    X = wl.X[rng.integers(0, wl.F, F)] + 0.1 * rng.standard_normal((F, 60)).astype(np.float32)
    X = dev(X.astype(np.float32))
    large, small = make_ctx(wl, max_frames=F), make_ctx(wl, max_frames=64)
    a, b = _lists(F), _lists(F)
    t_large = _ms(lambda: large.ubm_posteriors(X, post_idx=a[0], post_val=a[1], frame_ll=a[2],
                                               prec=prec))
    t_small = _ms(lambda: small.ubm_posteriors_static(X, *b, prec=prec))
    large.sync_status()
    small.sync_status()
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p.cpu().numpy(), q.cpu().numpy())
    assert t_small <= 4 * t_large, (t_small, t_large)


def test_static_call_beside_a_call_of_the_same_context():
    wl = synth.make(2, R=4, U=40, lengths="uniform:1000:1000")
    F = wl.F
    ctx = make_ctx(wl)
    X1, X2 = dev(wl.X), dev(wl.X[::-1])
    ref = []
    for X in (X1, X2):
        r = _lists(F)
        ctx.ubm_posteriors(X, post_idx=r[0], post_val=r[1], frame_ll=r[2])
        ctx.sync_status()
        ref.append([t.cpu().numpy() for t in r])
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(5):
        a, b = _lists(F), _lists(F)
        torch.cuda.synchronize()
        for _ in range(3):
            ctx.ubm_posteriors(X1, post_idx=a[0], post_val=a[1], frame_ll=a[2], stream=s1)
            ctx.ubm_posteriors_static(X2, *b, stream=s2)
        torch.cuda.synchronize()
        for out, want in zip((a, b), ref):
            for p, q in zip(out, want):
                np.testing.assert_array_equal(p.cpu().numpy(), q)
