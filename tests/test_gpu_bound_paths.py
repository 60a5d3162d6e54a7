"""The bound that preselects components in large batches, away from the workload's
models: against the dense kernel (an explicitly chosen launch shape), whose
candidate lists it has to leave bit for bit, and in its time, which shows how
many frames it had to hand on."""
import gc

import numpy as np
import pytest
import torch

import synth
from _gpu_helpers import dev

pytestmark = pytest.mark.gpu


def _frames(wl, F, seed):
    """F frames drawn from the workload's own, with noise; more than the score buffer holds."""
    rng = np.random.default_rng(seed)
    assert 4 * F * ((wl.shape.C + 255) // 256 * 256) > 64 << 20
    X = wl.X[rng.integers(0, wl.F, F)].astype(np.float64)
    return X + 0.1 * rng.standard_normal(X.shape)


def _context(w, mu, cov, F):
    from paper_1906_08556_amd import ivx
    ctx = ivx.Context(mu.shape[0], mu.shape[1], 2, 1, F)
    ctx.set_ubm(dev(w), dev(mu), dev(cov))
    return ctx


def _run(ctx, X, prec, ncb, timed=False, check=True):
    """Posterior lists with frame_ncb = ncb (8: the default route, 4: dense); least of 5 times."""
    F = X.shape[0]
    pi = torch.full((F, 16), -7, dtype=torch.int32, device="cuda")
    pv = torch.full((F, 16), -7.0, device="cuda")
    ll = torch.full((F,), -7.0, dtype=torch.float64, device="cuda")
    ctx.tuning_set(frame_ncb=ncb, frame_ncb_bf16=ncb)
    ms = []
    for _ in range(6 if timed else 1):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        ctx.ubm_posteriors(X, post_idx=pi, post_val=pv, frame_ll=ll, prec=prec)
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    if check:
        ctx.sync_status()
    return [t.cpu().numpy() for t in (pi, pv, ll)], min(ms)


def _same(a, b):
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("scale", [2.0 ** -8, 2.0 ** -4, 2.0 ** 9])
def test_bound_does_not_depend_on_the_scale_of_the_features(scale):
    """Scaled by a power of two every product of the bound is the same; the time
    is that of the unscaled model (factor 1.5: other work of the call is there
    too, and a frame handed on costs six times one that is not)."""
    wl = synth.make(2, R=4, U=20, lengths="uniform:1000:1000")
    X = _frames(wl, 60000, 1).astype(np.float32)
    plain = _context(wl.w, wl.mu, wl.cov, len(X))
    _, t0 = _run(plain, dev(X), 0, 8, timed=True)
    ctx = _context(wl.w, scale * wl.mu, scale ** 2 * wl.cov, len(X))
    Xs = dev((scale * X).astype(np.float32))
    got, t1 = _run(ctx, Xs, 0, 8, timed=True)
    _same(got, _run(ctx, Xs, 0, 4)[0])
    assert t1 <= 1.5 * t0, (t1, t0)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("offset", [-2.0 ** 13, 2.0 ** 20])
def test_bound_with_features_far_from_the_origin(offset, prec):
    """FP32 features at an offset are 2^-11 or 2^-4 apart, but exact inputs: the
    lists are those of the dense kernel, which takes them from their mean."""
    wl = synth.make(2, R=4, U=20, lengths="uniform:1000:1000")
    X = dev((_frames(wl, 30000, 2) + offset).astype(np.float32))
    ctx = _context(wl.w, wl.mu + offset, wl.cov, len(X))
    _same(_run(ctx, X, prec, 8)[0], _run(ctx, X, prec, 4)[0])


def test_padding_components_are_never_taken():
    """A model so wide that the scaled constants of its components (-2 S^2 cst_c,
    about 1e33) pass any finite constant of a padding component; every frame
    is within the margin of all of them and goes to the dense kernel."""
    C, D, F, wide = 700, 33, 30000, 2.0 ** 108
    rng = np.random.default_rng(3)
    w = np.full(C, 1.0 / C)
    mu = wide * rng.standard_normal((C, D))
    mu -= mu.mean(0)
    cov = np.broadcast_to(wide ** 2 * np.eye(D), (C, D, D)).copy()
    X = dev((1e3 * rng.standard_normal((F, D))).astype(np.float32))
    ctx = _context(w, mu, cov, F)
    a, _ = _run(ctx, X, 0, 8, check=False)
    assert a[0].max() < C
    _same(a, _run(ctx, X, 0, 4, check=False)[0])


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("C,D,std,shift", [(2048, 60, 6.0, 12.0), (2048, 40, 6.0, 12.0),
                                           (640, 60, 6.0, 12.0), (2048, 60, 4.0, 8.0),
                                           (2048, 32, 6.0, 12.0)])
def test_models_whose_components_the_bound_cannot_exclude(C, D, std, shift, prec):
    """Well-conditioned covariances (600 degrees of freedom) and frames far from all
    means: 32 rows see too little of the distances.  The lists are the dense
    kernel's and the call takes no longer than a dense shape (a quarter for timing
    and the launches that find nothing to do; with the sweeps wasted the BF16
    calls take half as long again)."""
    F = 36000
    rng = np.random.default_rng(D)
    w = rng.dirichlet(np.full(C, 5.0))
    mu = std * rng.standard_normal((C, D))
    cov = np.empty((C, D, D))
    for c in range(C):
        A = rng.standard_normal((600, D), dtype=np.float32).astype(np.float64)
        cov[c] = A.T @ A / 600
    X = (mu[rng.integers(0, C, F)] + shift * rng.standard_normal((F // 1000, D)).repeat(1000, 0)
         + rng.standard_normal((F, D)))
    X = dev(X.astype(np.float32))
    ctx = _context(w, mu, cov, F)
    got, t = _run(ctx, X, prec, 8, timed=True)
    want, t4 = _run(ctx, X, prec, 4, timed=True)
    _same(got, want)
    assert t <= 1.25 * t4, (t, t4)


def test_memory_of_a_context_with_many_components():
    """The sums between the sweeps take at most 2 GB, also where that holds fewer
    frames than the device works on (8192 < C); 1 KB per frame for all else."""
    from paper_1906_08556_amd import ivx

    gc.collect()  # contexts of other tests

    def used(F):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx = ivx.Context(16384, 32, 2, 1, F)
        n = free - torch.cuda.mem_get_info()[0]
        del ctx
        return n

    used(2000)  # the library's own first-time allocations
    assert used(140000) - used(2000) <= (2 << 30) + (64 << 20) + 1024 * 140000


@pytest.mark.parametrize("C,D,F,prec", [(512, 32, 33000, 0), (512, 40, 140000, 1), (701, 62, 22000, 0),
                                        (701, 62, 22000, 1), (2048, 33, 9000, 0)])
def test_bound_at_the_edges_of_its_range(C, D, F, prec):
    """Fewest components and dimensions, most dimensions, padded components, rows that
    are no whole float4: with lists that overflow (100 nearly equal components) and
    frames outside the bound's range, the lists are the dense kernel's."""
    from paper_1906_08556_amd import ivx
    wl = synth.make(2, C=C, D=D, R=4, U=20, lengths="uniform:1000:1000")
    X = _frames(wl, F, 6)
    mu, cov = wl.mu.copy(), wl.cov.copy()
    mu[-100:] = mu[-1] + 50.0 + 1e-3 * np.arange(100)[:, None]
    cov[-100:] = cov[-1]
    rng = np.random.default_rng(5)
    X[100:140] = mu[-50] + rng.standard_normal((40, D)) @ np.linalg.cholesky(cov[-1]).T
    X[200:210] *= 1e4
    X[300] = 3e7
    X[301, D - 1] = np.inf
    X[F - 1, 0] = np.nan
    X = dev(X.astype(np.float32))
    ctx = _context(wl.w, mu, cov, F)
    out = []
    for ncb in (8, 4):
        out.append(_run(ctx, X, prec, ncb, check=False)[0])
        with pytest.raises(ivx.IvxError):
            ctx.sync_status()
    assert np.all(out[0][0][100:140] >= C - 100)
    _same(*out)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
def test_more_frames_handed_on_than_the_score_buffer_holds(prec):
    """22,500 of 150,000 frames lie beyond the bound's range (2^21 units): the dense
    kernel takes them through their list, and the others' lists are its own too."""
    wl = synth.make(2, R=4, U=20, lengths="uniform:1000:1000")
    X = _frames(wl, 150000, 7)
    X[np.random.default_rng(8).permutation(len(X))[:22500]] *= 1e7
    X = dev(X.astype(np.float32))
    ctx = _context(wl.w, wl.mu, wl.cov, len(X))
    _same(_run(ctx, X, prec, 8)[0], _run(ctx, X, prec, 4)[0])


def test_bound_of_two_contexts_on_two_streams():
    wl = synth.make(2, R=4, U=20, lengths="uniform:1000:1000")
    X = [dev(_frames(wl, 30000, s).astype(np.float32)) for s in (9, 10)]
    ctx = [_context(wl.w, wl.mu, wl.cov, 30000) for _ in X]
    want = [_run(c, x, 0, 8)[0] for c, x in zip(ctx, X)]
    streams = [torch.cuda.Stream() for _ in X]
    for _ in range(5):
        out = [(torch.full((30000, 16), -7, dtype=torch.int32, device="cuda"),
                torch.full((30000, 16), -7.0, device="cuda"),
                torch.full((30000,), -7.0, dtype=torch.float64, device="cuda")) for _ in X]
        torch.cuda.synchronize()
        for c, x, o, s in zip(ctx, X, out, streams):
            c.ubm_posteriors(x, post_idx=o[0], post_val=o[1], frame_ll=o[2], stream=s)
        torch.cuda.synchronize()
        for o, w in zip(out, want):
            _same([t.cpu().numpy() for t in o], w)
