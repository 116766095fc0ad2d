"""Candidate masks where their computation has edges: tools that share them (the
same directions and arm samples) scored together against each scored alone, at
orientation counts round the mask words and the four words of a launch, and a
map with more points than the kernel for small maps takes against the oracle.
Masks, labels and statistics are whole numbers and must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STATS = ("n_points", "n_confident", "n_accessible", "n_blocked", "n_no_candidate", "candidate_tests",
         "canonical_tests", "canonical_lookups", "arm_lookups")


def results(ctx, tool):
    lab, st, dbg = ctx.read_labels(tool), ctx.score_stats(tool), ctx.read_point_debug(tool)
    return [lab["label"], lab["first_free"], dbg["mask"], [st[k] for k in STATS]]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def rotations(rng, n_dirs, n_roll):
    """n_roll rotations about each of n_dirs random directions (roll-minor)."""
    out = []
    for _ in range(n_dirs):
        x = rng.normal(size=3)
        x /= np.linalg.norm(x)
        u = np.cross(x, (0.3, 0.5, 0.8))
        u /= np.linalg.norm(u)
        v = np.cross(x, u)
        for r in range(n_roll):
            c, s = np.cos(np.pi * r / n_roll), np.sin(np.pi * r / n_roll)
            out.append(np.stack([x, c * u + s * v, c * v - s * u], 1))
    return np.array(out)


@pytest.mark.parametrize("n_dirs,n_roll", [(1, 1), (16, 4), (65, 1), (97, 3), (257, 1), (128, 4)])
def test_shared_masks(synth_mod, n_dirs, n_roll):
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17,
                                 max_orientations=512, max_tools=4))
    for f in w.frames(6):
        ctx.integrate_frame(torch.from_numpy(f.xyz).cuda(), f.origin, f.frame_id)
    rng = np.random.default_rng(n_dirs)
    rot, other = rotations(rng, n_dirs, n_roll), rotations(rng, n_dirs, n_roll)
    tool = w.tool
    ctx.set_tool_kernels(0, tool, rot)
    ctx.set_tool_kernels(1, tool, other)   # other directions
    ctx.set_tool_kernels(2, synth_mod.box_tool(corridor=0.5), rot)
    ctx.set_tool_kernels(3, tool, other)
    ctx.set_tool_kernels(3, tool, rot)     # loaded anew: shares with 0 now
    alone = []
    for t in range(4):
        ctx.score_points(t)
        alone.append(results(ctx, t))
    ctx.score_tools([0, 1, 2, 3])
    for t in range(4):
        assert same(results(ctx, t), alone[t]), t
    assert not np.array_equal(alone[0][2], alone[1][2])
    ctx.score_tools([3, 1])
    for t in (1, 3):
        assert same(results(ctx, t), alone[t]), t


def test_many_points(oracle_mod, synth_mod):
    """300,000 points: one wave per 64 points."""
    import torch
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    voxel, trunc = 0.01, 0.02
    ctx = Context(default_config(voxel, trunc, r_c=0.005, max_blocks=1 << 15, max_points=1 << 19,
                                 max_orientations=128, max_tools=1))
    orc = oracle_mod.Oracle(voxel=voxel, trunc=trunc, r_c=0.005)
    rng = np.random.default_rng(4)
    for i in range(3):
        xyz = rng.uniform((-4.0, -4.0, 0.0), (4.0, 4.0, 0.004), (160000, 3)).astype(np.float32)
        q = np.array([0.5 * i, 0.1, 1.5], np.float32)
        ctx.integrate_frame(torch.from_numpy(xyz).cuda(), q, i)
        orc.integrate_frame(xyz, q, i)
    rot = rotations(rng, 23, 3)
    ctx.set_tool_kernels(0, w.tool, rot)
    orc.set_tool(0, w.tool, rot)
    ctx.score_points(0)
    orc.score(0)
    assert ctx.num_points() > 262144
    key = ctx.read_points()["key"]
    dbg = ctx.read_point_debug(0)
    for i in rng.integers(len(key), size=400):
        r = orc.point_result(key[i], len(rot))
        assert np.array_equal(dbg["mask"][i], r["mask"]), i
    g, o = ctx.score_stats(0), orc.score_stats()
    for k in ("n_points", "n_confident", "n_accessible", "n_blocked", "n_no_candidate", "candidate_tests",
              "canonical_tests", "canonical_lookups"):
        assert g[k] == o[k], k
