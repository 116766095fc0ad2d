"""GPU parity of the chunk scan (the default scoring configuration) against the
plain one, which tests a table entry by entry, at the sizes where the chunk
form can go wrong: class sizes round multiples of 64 and above 64 and 128
corridor chunks, orientation counts round a mask word and the staged first
chunks, offsets at and above the largest the form takes, the point list, the
few-points deal and several tools in one launch.  Labels, first free
orientations and statistics are whole numbers and must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BODY, NEAR, FAR = 0, 1, 2
STATS = ("n_points", "n_confident", "n_accessible", "n_blocked", "n_no_candidate", "candidate_tests",
         "canonical_tests", "canonical_lookups")


@pytest.fixture(scope="module")
def tiny_map(synth_mod):
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    cfg = default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17,
                         max_orientations=512, max_tools=2)
    ctx = Context(cfg)
    for f in w.frames():
        ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
    return ctx


def make_table(K, body, far, reach, seed=3):
    """K orientations along random directions: `body` entries round the arm,
    `far` in a thin rod beyond it, the furthest at `reach` voxels on an axis."""
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(K, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    d[0] = (1.0, 0.0, 0.0)
    begin, off, cls = [0], [], []
    for ax in d:
        near = np.rint(np.array([[2.0], [4.0], [7.0]]) * ax).astype(np.int64)
        taken = {tuple(o) for o in near} | {(0, 0, 0)}
        rows = [(o, NEAR) for o in near]
        u = np.cross(ax, (0.3, 0.5, 0.8))
        u /= np.linalg.norm(u)
        v = np.cross(ax, u)
        for c, n, lo, hi in ((BODY, body, 3.0, 30.0), (FAR, far, 32.0, reach - 1.0)):
            want = len(rows) + n
            if n and c == FAR:
                rows.append((np.array([reach, 0, 0]), FAR))
                taken.add((reach, 0, 0))
            while len(rows) < want:
                t, a, b = rng.uniform((lo, -5.0, -5.0), (hi, 5.0, 5.0))
                o = np.rint(t * ax + a * u + b * v).astype(np.int64)
                if abs(o).max() <= reach and tuple(o) not in taken:
                    taken.add(tuple(o))
                    rows.append((o, c))
        off += [o for o, _ in rows]
        cls += [c for _, c in rows]
        begin.append(len(off))
    return d, np.array(begin, np.uint32), np.array(off, np.int16), np.array(cls, np.uint8)


def results(ctx, tool):
    lab, st = ctx.read_labels(tool), ctx.score_stats(tool)
    return lab["label"], lab["first_free"], [st[k] for k in STATS]


def same(a, b):
    return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]


# body and corridor sizes round one and several chunks, no body, no corridor,
# 65 and 129 corridor chunks (groups of 1, 2 and 4); K round a mask word, the
# staged first chunks (256) and above; reach round the largest taken (255)
@pytest.mark.parametrize("K,body,far,reach", [
    (1, 1, 0, 40), (1, 0, 1, 41), (2, 0, 0, 9), (63, 63, 64, 60), (64, 64, 65, 90), (65, 65, 63, 90),
    (129, 127, 129, 120), (256, 128, 192, 120), (257, 129, 193, 120), (291, 192, 320, 247),
    (3, 40, 4097, 254), (2, 70, 8193, 255), (2, 70, 128, 256)])
def test_chunks_against_plain(tiny_map, K, body, far, reach):
    ctx = tiny_map
    table = make_table(K, body, far, reach)
    ctx.set_tool_table(0, *table)
    best = ctx.score_variant_default()
    out = []
    for v in (best, 0):
        ctx.set_score_variant(v)
        ctx.score_points(0)
        out.append(results(ctx, 0))
    ctx.set_score_variant(best)
    assert out[0][2][0] > 0
    assert out[0][2] == out[1][2]
    assert same(out[0], out[1])
    # with a second tool in one launch
    ctx.set_tool_table(1, *make_table(5, 80, 200, 100, seed=4))
    ctx.score_points(1)
    single = results(ctx, 1)
    ctx.score_tools([0, 1])
    assert same(results(ctx, 0), out[1])
    assert same(results(ctx, 1), single)


def test_chunk_tables_make_room(synth_mod):
    """A context whose memory budget leaves no room for the chunk tables still
    loads and scores its tools, and a later allocation takes their room."""
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    frames = w.frames()

    table = make_table(16, 100, 1000, 120)

    def load(budget):
        ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17,
                                     max_orientations=64, max_tools=1, hbm_budget=budget))
        ctx.set_tool_table(0, *table)
        return ctx

    def score(ctx):
        for f in frames:
            ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
        ctx.score_points(0)
        return results(ctx, 0)

    ctx = load(0)
    loaded = ctx.device_bytes()
    free, end = score(ctx), ctx.device_bytes()
    assert load(loaded - 1).device_bytes() < loaded - 1
    ctx = load(end - 1)
    assert same(score(ctx), free) and ctx.device_bytes() < end - 1
