"""GPU tests of a memory budget that does not hold the grid: what the call that
failed had allocated is given back, and once there is room the context goes on
with the results of one without a budget (whole numbers, equal)."""
import dataclasses

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
    _, ref = context(synth_mod, 0)
    integrate(ref, f)
    ref.set_tool_kernels(0, w.tool, w.rot)
    assert ctx.device_bytes() == ref.device_bytes()
    ctx.score_points(0)
    assert scores(ctx) == want


def far_frame(synth_mod, w, i, far=2.0):
    """Frame i with returns `far` metres away on every side, three times each."""
    f = w.frames(i + 1)[i]
    d = np.concatenate([np.eye(3), -np.eye(3)]).astype(np.float32) * np.float32(far)
    return dataclasses.replace(f, xyz=np.concatenate([f.xyz, d, d, d]).astype(np.float32))


def same_map(a, b):
    for x, y in zip(a.read_tsdf(), b.read_tsdf()):
        assert np.array_equal(x, y)
    pa, pb = a.read_points(), b.read_points()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]), k


# again: the refused frame is given a second time once there is room; else the
# frames go on without it
@pytest.mark.parametrize("window", [None, (40, 40, 40)])
@pytest.mark.parametrize("again", [True, False])
def test_frames_go_on_after_a_refused_one(synth_mod, again, window):
    from paper_2608_06412_amd import AFError
    sizes = dict(max_orientations=1025, max_tools=2)
    large = synth_mod.cylinder_tool(0.06, 0.1, 1.0)   # (1,025 orientations: no chunk tables)
    many = synth_mod.orientations(synth_mod.fibonacci_directions(1025), 1)

    def load(budget):
        w, ctx = context(synth_mod, budget, **sizes)
        ctx.set_tool_kernels(0, w.tool, w.rot)
        return w, ctx

    w, ctx = load(0)
    frames = w.frames(5)
    # without a window frame 1 makes the grid grow; a window's first frame makes its grid
    stop = 0 if window else 1
    frames[stop] = far_frame(synth_mod, w, stop)
    loaded = ctx.device_bytes()
    tables = loaded - load(loaded - 1)[1].device_bytes()
    assert tables > 0

    def prepare(ctx):
        if window:
            ctx.set_window(window)
        ctx.set_tool_kernels(1, large, many)
        for f in frames[:stop]:
            integrate(ctx, f)

    prepare(ctx)
    integrate(ctx, frames[stop])
    end = ctx.device_bytes()
    del ctx
    w, ctx = load(end - tables - 1)
    prepare(ctx)
    for _ in range(2):
        with pytest.raises(AFError) as e:
            integrate(ctx, frames[stop])
        assert e.value.code == ENOMEM
    assert ctx.num_points() == (0 if window else len(np.unique(ctx.read_points()["key"])))
    ctx.set_tool_kernels(1, w.tool, w.rot[:2])        # room
    w, ref = load(0)
    if window:
        ref.set_window(window)
    ref.set_tool_kernels(1, w.tool, w.rot[:2])
    for i, f in enumerate(frames):
        if i >= stop + (not again):
            integrate(ctx, f)
        if not again and i == stop:   # (it has placed the window)
            f = dataclasses.replace(f, xyz=f.xyz[:0])
        integrate(ref, f)
    assert not again or ctx.num_blocks() == ref.num_blocks()
    same_map(ctx, ref)
    for c in (ctx, ref):
        c.score_points(0)
    assert scores(ctx) == scores(ref)
    assert ref.score_stats(0)["n_confident"] > 100


def test_refused_frame_leaves_the_map_as_it_was(synth_mod):
    """Without a budget: no grid covers returns 900 m away."""
    from paper_2608_06412_amd import AFError
    w, ctx = context(synth_mod, 0)
    _, ref = context(synth_mod, 0)
    f = w.frames(3)
    for c in (ctx, ref):
        integrate(c, f[0])
        integrate(c, f[1])
    for _ in range(3):
        with pytest.raises(AFError) as e:
            integrate(ctx, far_frame(synth_mod, w, 2, 900.0))
        assert e.value.code == ENOMEM
        same_map(ctx, ref)
    with pytest.raises(AFError):
        integrate(ctx, f[1])      # (ids increase)
