"""The incremental mode's sample of changed voxels and its count of raw
collisions where their paths change: frames of a few returns (all changed
voxels sampled; up to 1,024; up to 2,048, which the sort goes through itself;
more, through the first bound), an empty one and a full one, against the
oracle's state machine.  Everything is a whole number or an exact replay and
must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STATS = ("trig_i", "trig_ii", "trig_iii", "sampled", "evaluated", "backlog")


@pytest.mark.parametrize("budget", [100, 100000])
def test_sample_sizes(synth_mod, oracle_mod, budget):
    import torch
    from oracle.incremental import IncrementalOracle
    from paper_2608_06412_amd import Context, default_config
    w = synth_mod.tiny()
    full = w.frames(14)
    ctx = Context(default_config(w.voxel, w.trunc, r_c=w.r_c, max_blocks=1 << 15, max_points=1 << 17))
    ctx.set_tool_kernels(0, w.tool, w.rot)
    ctx.incremental_enable(0, budget)
    orc = oracle_mod.Oracle(voxel=w.voxel, trunc=w.trunc, r_c=w.r_c)
    orc.set_tool(0, w.tool, w.rot)
    inc = IncrementalOracle(orc, 0, len(w.rot), budget=budget)
    seen = set()
    counts = (2000, 2000, 1, 0, 2, 3, 4, 5, 6, 7, 9, 12, 40, 2000)
    for f, n in zip(full, counts):
        xyz = np.ascontiguousarray(f.xyz[:n])
        ctx.incremental_frame(torch.from_numpy(xyz).cuda(), f.origin, f.frame_id)
        ost = inc.frame(xyz, f.origin, f.frame_id)
        gst = ctx.incremental_stats()
        assert {k: gst[k] for k in STATS} == {k: ost[k] for k in STATS}, n
        changed = ctx.frame_stats()["voxels_folded"]
        seen.add("all" if changed <= 1024 else "sort" if changed <= 2048 else "bound")
        g = ctx.read_incremental()
        keys, lab, best, bdir, a = inc.labels()
        assert np.array_equal(g["key"], keys) and np.array_equal(g["label"], lab), n
        assert np.array_equal(g["best"].astype(np.int32), best), n
        assert np.array_equal(g["best_dir"].astype(np.int32), bdir) and np.array_equal(g["a"], a), n
    assert seen == {"all", "sort", "bound"}
