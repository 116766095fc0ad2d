"""GPU parity of the binned integration against the CPU oracle where its split
of the work has edges: returns per frame round a wave, returns per block round
the waves of a workgroup, a batch of 512 and a pass of 1,023, cubes from one
to fifteen voxels wide (with and without the negative clamp), returns on voxel
centres and corners, more new points than one round of the append's waves,
repeated frames on touched blocks, and dropped returns between valid ones.
Everything is a whole number and must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STATS = ("n_in", "n_valid", "n_dropped", "pairs_applied", "pairs_excluded", "band_marks", "new_points",
         "n_points", "voxels_folded")
VOXEL = 0.01


def same_maps(ctx, orc):
    for a, b, name in zip(ctx.read_tsdf(), orc.read_tsdf(), ("key", "S", "W", "cleared")):
        assert np.array_equal(np.asarray(a, np.int64), np.asarray(b, np.int64)), name
    g, o = ctx.read_points(), orc.read_points()
    for name in ("key", "first_frame", "n_vp", "vp", "sumq", "nq"):
        assert np.array_equal(g[name], o[name]), name


def frames_of(kind, n, rng):
    """Two frames of n returns each (float32) with their sensor origins."""
    out = []
    for f in range(2):
        if kind == "block":      # all in one or two blocks
            xyz = rng.uniform(0.001, 0.099, (n, 3))
        elif kind == "lattice":  # voxel centres and corners, axis-parallel rays among them
            xyz = rng.integers(-20, 20, (n, 3)) * (VOXEL / 2)
        else:                    # spread over many blocks
            xyz = rng.uniform(-1.0, 1.0, (n, 3)) * (1.0, 1.0, 0.2)
        if kind == "dropped":
            xyz[::3] = np.nan
            xyz[1::7] = (0.3, 0.2, 1.5)   # the sensor itself
        q = (0.3, 0.2, 1.5) if kind != "lattice" else (0.0, 0.0, 1.5)
        out.append((xyz.astype(np.float32), np.array(q, np.float32)))
    return out


@pytest.mark.parametrize("kind,n,R", [
    ("block", 1, 1), ("block", 7, 1), ("block", 9, 3), ("block", 64, 4), ("block", 65, 5), ("block", 511, 4),
    ("block", 513, 4), ("block", 1023, 3), ("block", 1025, 4), ("block", 2300, 7), ("lattice", 300, 4),
    ("lattice", 700, 6), ("spread", 63, 2), ("spread", 129, 7), ("spread", 6000, 4), ("dropped", 500, 4)])
@pytest.mark.parametrize("clamp_neg", [0, 1])
def test_integration_at_edges(oracle_mod, kind, n, R, clamp_neg):
    import torch
    from paper_2608_06412_amd import Context, default_config
    trunc = R * VOXEL
    ctx = Context(default_config(VOXEL, trunc, max_blocks=1 << 14, max_points=1 << 15, max_orientations=64,
                                 max_tools=1, clamp_negative=clamp_neg))
    orc = oracle_mod.Oracle(voxel=VOXEL, trunc=trunc, clamp_negative=clamp_neg)
    for i, (xyz, q) in enumerate(frames_of(kind, n, np.random.default_rng(n))):
        ctx.integrate_frame(torch.from_numpy(xyz).cuda(), q, i)
        orc.integrate_frame(xyz, q, i)
        g, o = ctx.frame_stats(), orc.frame_stats()
        assert {k: g[k] for k in STATS} == {k: o[k] for k in STATS}
        same_maps(ctx, orc)
