"""GPU tests of a memory budget that makes an allocation take the room of the
tools' chunk tables in the middle of a call.  Wherever in the call that
happens, labels, first free orientations and statistics are those of a context
without a budget (whole numbers, equal)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

IDS = [0, 1]


def load(synth_mod, budget):
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 13, max_points=1 << 14,
                                 max_orientations=256, max_tools=2, hbm_budget=budget))
    for i in IDS:
        ctx.set_tool_kernels(i, synth_mod.cylinder_tool(0.06 - 0.01 * i, 0.3, 1.0),
                             synth_mod.orientations(synth_mod.fibonacci_directions(128 + 2 * i), 1))
    return w, ctx


def mapped(synth_mod, budget):
    import torch
    w, ctx = load(synth_mod, budget)
    for f in w.frames(4):
        ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
    return ctx


def results(ctx, ids):
    out = []
    for i in ids:
        lab = ctx.read_labels(i)
        out.append((lab["label"].tolist(), lab["first_free"].tolist(), ctx.score_stats(i)))
    return out


@pytest.mark.parametrize("ids", [[0], [0, 1], [1, 0]])
def test_dropped_inside_score_tools(synth_mod, ids):
    ctx = mapped(synth_mod, 0)
    before = ctx.device_bytes()
    ctx.score_tools(ids)
    want, end = results(ctx, ids), ctx.device_bytes()
    assert 1 in want[0][0] and 2 in want[0][0]
    ctx = mapped(synth_mod, end - 1)     # the call's last allocation takes the tables' room
    assert ctx.device_bytes() == before
    ctx.score_tools(ids)
    tables = end - ctx.device_bytes()
    assert tables > 1 << 20
    assert results(ctx, ids) == want
    # ... and the others down to the first that still leaves the call enough
    for budget in np.linspace(max(before, end - tables), end - 1, 7).astype(np.int64)[:-1]:
        ctx = mapped(synth_mod, int(budget))
        print("budget", budget, "of", end, flush=True)
        ctx.score_tools(ids)
        assert ctx.device_bytes() == end - tables
        assert results(ctx, ids) == want
        ctx.score_points(ids[-1])        # and the next calls
        ctx.score_tools(ids)
        assert results(ctx, ids) == want


def test_kept_when_their_room_is_not_enough(synth_mod):
    """A call that does not fit even in the tables' room is refused and leaves
    them; one that does takes it."""
    from paper_2608_06412_amd import AFError
    ctx = mapped(synth_mod, 0)
    ctx.score_points(0)
    held, want = ctx.device_bytes(), results(ctx, [0])
    ctx = mapped(synth_mod, held)
    ctx.score_points(0)
    for n in (1 << 21, 1 << 22):
        with pytest.raises(AFError) as e:
            ctx.integrate_frame(np.zeros((n, 3), np.float32), np.zeros(3, np.float32), 100)
        assert e.value.code == -2
        assert ctx.device_bytes() == held
    ctx.score_points(0)
    assert results(ctx, [0]) == want
    ctx.integrate_frame(np.zeros((1500, 3), np.float32), np.zeros(3, np.float32), 100)
    assert ctx.device_bytes() < held
    ctx.score_points(0)
    assert results(ctx, [0]) == want


@pytest.mark.parametrize("ids", [[0], [0, 1]])
def test_recorded_frames_go_on_after_a_drop(synth_mod, ids):
    import torch
    w = synth_mod.tiny()
    frames = w.frames(8)
    xs = [torch.from_numpy(f.xyz).cuda() for f in frames]
    rng = np.random.default_rng(3)
    p = torch.from_numpy(rng.uniform(-1, 1, (500, 3)).astype(np.float32)).cuda()
    q = torch.from_numpy(rng.normal(size=(500, 4)).astype(np.float32)).cuda()
    samples = torch.from_numpy(np.ascontiguousarray(
        synth_mod.tool_samples(synth_mod.cylinder_tool(), 16), np.float32)).cuda()

    def smooth(ctx):
        s = torch.empty(len(p), device="cuda")
        ctx.smooth_eval(p, q, samples, 0.01, 0.005, s=s)
        return s.cpu().numpy()

    def run(budget):
        _, ctx = load(synth_mod, budget)
        ctx.graph_prepare([-3, -3, -1], [3, 3, 3], len(xs[0]), ids)
        out, held = [], []
        for j, f in enumerate(frames):
            if j == 4:
                held.append(ctx.device_bytes())
                out.append(smooth(ctx))
                held.append(ctx.device_bytes())
            ctx.graph_frame(xs[j], f.origin, f.frame_id)
            if j % 2:
                ctx.graph_sync()
                out.append(results(ctx, ids))
        return ctx, out, held

    _, want, held = run(0)
    ctx, got, tight = run(held[1] - 1)
    assert tight[0] == held[0] and tight[1] < held[1] - (1 << 20)
    for a, b in zip(got, want):
        assert np.array_equal(a, b) if isinstance(a, np.ndarray) else a == b
    _, eager = load(synth_mod, 0)
    for x, f in zip(xs, frames):
        eager.integrate_frame(x, f.origin, f.frame_id)
    eager.score_tools(ids)
    assert results(eager, ids) == got[-1]


def test_refused_by_the_device_is_no_later_error(synth_mod):
    """A device allocation that fails is reported by its call, not by the next
    launch (a context goes on, where it can, without what it did not get)."""
    import torch
    from paper_2608_06412_amd import AFError
    ctx, ref = mapped(synth_mod, 0), mapped(synth_mod, 0)
    with pytest.raises(AFError) as e:
        ctx.graph_prepare([-3, -3, -1], [3, 3, 3], 1 << 40, [0])   # 16 TiB of scratch
    assert e.value.code == -2
    f = synth_mod.tiny().frames(6)[5]
    for c in (ctx, ref):
        c.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
        c.score_tools(IDS)
    assert results(ctx, IDS) == results(ref, IDS)
