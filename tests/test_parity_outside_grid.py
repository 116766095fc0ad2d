"""GPU tests of points that lie outside the grid of a recorded frame: the frame
maps and scores them before the host hears of it.  It is reported, the scoring
reads nothing outside the grid's planes (their far points get a label from the
arm samples and an empty plane), and eager frames go on as in a context that
never recorded one.  A block that comes nearer to the grid's border than a tool
loaded later reaches is reported as well."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def make(synth_mod, n_tools):
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17,
                                 max_orientations=512, max_tools=n_tools))
    return w, ctx


def with_far(xyz, far):
    """The frame's returns and, three times each, returns `far` metres away."""
    d = np.array([[1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1],
                  [-1, -1, -1], [1, 1, 1]], np.float32) * np.float32(far)
    return np.concatenate([xyz, d, d, d]).astype(np.float32)


@pytest.mark.parametrize("far", [2.0, 6.0, 900.0])
@pytest.mark.parametrize("n_tools", [1, 2])
def test_recorded_points_outside(synth_mod, far, n_tools):
    import torch
    from paper_2608_06412_amd import AFError
    ids = list(range(n_tools))
    w, rec = make(synth_mod, n_tools)
    _, eager = make(synth_mod, n_tools)
    for ctx in (rec, eager):
        for i in ids:
            ctx.set_tool_kernels(i, w.tool, w.rot[:64 - 3 * i])
    frames = w.frames(3)
    o = np.asarray(frames[0].origin, np.float64)
    x0 = torch.from_numpy(with_far(frames[0].xyz, far)).cuda()
    rec.graph_prepare(o - 0.05, o + 0.05, len(x0), ids)
    rec.graph_frame(x0, frames[0].origin, frames[0].frame_id)
    with pytest.raises(AFError):
        rec.graph_sync()
    for i in ids:
        lab = rec.read_labels(i)
        assert set(np.unique(lab["label"])) <= {0, 1, 2, 3}
        assert rec.score_stats(i)["n_confident"] == int((lab["label"] != 0).sum()) >= 8
    if far > 10.0:   # (no grid covers that)
        return
    eager.integrate_frame(x0, frames[0].origin, frames[0].frame_id)
    for f in frames[1:]:
        x = torch.from_numpy(f.xyz).cuda()
        for ctx in (rec, eager):
            ctx.integrate_frame(x, f.origin, f.frame_id)
    for ctx in (rec, eager):
        ctx.score_tools(ids)
    for i in ids:
        a, b = rec.read_labels(i), eager.read_labels(i)
        for k in ("key", "label", "first_free"):
            assert np.array_equal(a[k], b[k]), (i, k)
        assert rec.score_stats(i) == eager.score_stats(i)


def test_margin_follows_the_tools(synth_mod):
    import torch
    from paper_2608_06412_amd import AFError
    w, ctx = make(synth_mod, 1)
    bs = 8 * w.voxel
    f = w.frames(1)[0]
    lo, hi = np.full(3, -50 * bs), np.full(3, 49.5 * bs)   # 100 blocks, 25 more on each side
    ctx.set_tool_kernels(0, synth_mod.cylinder_tool(), w.rot)            # reaches 30 voxels
    ctx.graph_prepare(lo, hi, 100000, [0])
    ctx.set_tool_kernels(0, synth_mod.cylinder_tool(corridor=2.5), w.rot)  # 130: 18 bricks
    ctx.graph_prepare(lo, hi, 100000, [0])
    near = np.repeat(np.array([[62.5 * bs, 0, 0]], np.float32), 3, axis=0)   # 12 blocks to the border
    ctx.graph_frame(torch.from_numpy(f.xyz).cuda(), f.origin, 1)
    ctx.graph_sync()
    ctx.graph_frame(torch.from_numpy(near).cuda(), f.origin, 2)
    with pytest.raises(AFError):
        ctx.graph_sync()
    ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, 3)
    ctx.score_points(0)
    assert ctx.score_stats(0)["n_confident"] > 0
