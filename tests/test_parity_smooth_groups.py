"""The smoothed score takes pairs in groups (four to a wave, fewer where there
are few pairs) and keeps a sample's cell from one ascent step to the next.
Neither may show: a pair evaluated or refined among n others gives bit for bit
what it gives alone, at counts round the group, the wave count and a second
round of the waves, and with sample counts below, at and above a wave.  The
sums are formed in the same order in either case, so nothing is tolerated."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

C, TS = 0.01, 0.005


@pytest.fixture(scope="module")
def tiny_map(synth_mod):
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17))
    for f in w.frames():
        ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
    return w, ctx


def evaluate(ctx, p, q, smp):
    import torch
    s, dq, dp = (torch.empty((len(p),) + k, device="cuda") for k in ((), (4,), (3,)))
    ctx.smooth_eval(p, q, smp, C, TS, s=s, dq=dq, dp=dp)
    only = torch.empty(len(p), device="cuda")
    ctx.smooth_eval(p, q, smp, C, TS, s=only)
    return [x.cpu().numpy() for x in (s, dq, dp, only)]


@pytest.mark.parametrize("n,M", [(1, 64), (2, 1), (3, 63), (5, 64), (1025, 65), (3073, 64), (20001, 64), (60002, 7)])
def test_pair_among_others(tiny_map, n, M):
    import torch
    w, ctx = tiny_map
    rng = np.random.default_rng(n)
    base = rng.uniform(-0.6, 0.6, (n, 3)) + (0.0, 0.0, 0.5)
    p = torch.from_numpy((base + rng.uniform(-0.02, 0.02, (n, 3))).astype(np.float32)).cuda()
    q = torch.from_numpy(rng.normal(size=(n, 4)).astype(np.float32)).cuda()
    smp = torch.from_numpy(rng.uniform((0, -0.03, -0.03), (0.5, 0.03, 0.03), (M, 3)).astype(np.float32)).cuda()
    full = evaluate(ctx, p, q, smp)
    assert np.isfinite(full[0]).all() and (n < 5 or np.ptp(full[0]) > 0)
    kw = dict(steps=7, eta=1e-3, max_step=0.05, c=C, tau_s=TS)
    up = [x.cpu().numpy() for x in ctx.smooth_refine(p, q, smp, **kw)]
    for i in np.unique(np.r_[0, n - 1, rng.integers(n, size=12)]):
        one = evaluate(ctx, p[i:i + 1], q[i:i + 1], smp)
        for a, b in zip(full, one):
            assert np.array_equal(a[i], b[0]), i
        ref = ctx.smooth_refine(p[i:i + 1], q[i:i + 1], smp, **kw)
        for a, b in zip(up, ref):
            assert np.array_equal(a[i], b.cpu().numpy()[0]), i
