"""The smoothed score of points so far away that their voxel coordinates leave
32 bits: no sample meets a mapped cell, so a pair scores what one that lies
just outside the map does, bit for bit, with gradients of zero; the pairs
beside it keep their values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

C, TS = 0.01, 0.005


@pytest.mark.parametrize("M", [1, 64, 130])
@pytest.mark.parametrize("far", [1e8, 1e9, 3e18, 3e30])
def test_far_pairs(synth_mod, far, M):
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17))
    for f in w.frames(4):
        ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
    rng = np.random.default_rng(M)
    sign = np.array([[x, y, z] for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)], np.float64)
    near = rng.uniform(-0.6, 0.6, sign.shape) + (0.0, 0.0, 0.5)
    q = rng.normal(size=(2 * len(sign), 4)).astype(np.float32)
    q[1::4] = (1, 0, 0, 0)
    smp = torch.from_numpy(rng.uniform((0, -0.03, -0.03), (0.5, 0.03, 0.03), (M, 3)).astype(np.float32)).cuda()

    def pairs(there):
        p = np.empty((2 * len(sign), 3))
        p[0::2], p[1::2] = near, np.where(sign == 0, near, there * sign)
        p[1::2][(sign == 0).all(1)] = there
        return torch.from_numpy(p.astype(np.float32)).cuda()

    def run(p):
        s, dq, dp = (torch.empty((len(p),) + k, device="cuda") for k in ((), (4,), (3,)))
        qd = torch.from_numpy(q).cuda()
        ctx.smooth_eval(p, qd, smp, C, TS, s=s, dq=dq, dp=dp)
        r = ctx.smooth_refine(p, qd, smp, steps=3, eta=1e-3, max_step=0.05, c=C, tau_s=TS)
        return [x.cpu().numpy() for x in (s, dq, dp, *r)]

    got, want = run(pairs(far)), run(pairs(50.0))
    assert np.isfinite(want[0]).all() and np.ptp(want[0]) > 0
    assert (want[1][1::2] == 0).all() and (want[2][1::2] == 0).all()
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
