"""GPU tests of a memory budget that does not hold the grid: what the call that
failed had allocated is given back, and once there is room the context goes on
with the results of one without a budget (whole numbers, equal)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ENOMEM = -2


def context(synth_mod, budget, **sizes):
    import torch  # noqa: F401  (before the library: its HIP runtime serves both)
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    return w, Context(default_config(w.voxel, w.trunc, r_c=w.r_c, hbm_budget=budget,
                                     **{**dict(max_blocks=1 << 13, max_points=1 << 14,
                                               max_orientations=64, max_tools=1), **sizes}))


def integrate(ctx, f, fid=None):
    import torch
    ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id if fid is None else fid)


def scores(ctx, tool=0):
    lab = ctx.read_labels(tool)
    return [lab[k].tolist() for k in ("key", "label", "first_free")], ctx.score_stats(tool)


def test_failed_growth_gives_its_planes_back(synth_mod):
    from paper_2608_06412_amd import AFError
    far = synth_mod.cylinder_tool(corridor=6.0)   # reaches 305 voxels: 40 bricks of margin
    w, ctx = context(synth_mod, 0)
    f = w.frames(1)[0]
    integrate(ctx, f)
    ctx.set_tool_kernels(0, far, w.rot[:2])
    end = ctx.device_bytes()
    ctx.set_tool_kernels(0, w.tool, w.rot)
    ctx.score_points(0)
    want = scores(ctx)
    w, ctx = context(synth_mod, end - 1)
    integrate(ctx, f)
    held = []
    for _ in range(3):
        with pytest.raises(AFError) as e:
            ctx.set_tool_kernels(0, far, w.rot[:2])
        assert e.value.code == ENOMEM
        held.append(ctx.device_bytes())
    assert held[0] == held[1] == held[2]
    ctx.set_tool_kernels(0, w.tool, w.rot)
    ctx.score_points(0)
    assert scores(ctx) == want
