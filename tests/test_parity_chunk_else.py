"""GPU parity where the chunk scan cannot run: a flat map so wide that its grid
is beyond the scan's 32-bit offsets (60 m square at 1 cm).  The default
configuration then runs the staged entry scan, with up to 256 orientations, and
the entry scan above; labels, first free orientations and statistics equal the
plain configuration's, for one tool and for several in one launch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def patch(rng, at, n=3000):
    """Returns on an upright cross of two boards that stand `at`."""
    u = rng.uniform(-0.15, 0.15, (n, 2))
    p = np.zeros((n, 3))
    p[: n // 2, 0], p[n // 2:, 1] = u[: n // 2, 0], u[n // 2:, 0]
    p[:, 2] = u[:, 1]
    return p + np.asarray(at)


def test_flat_map_against_plain(synth_mod):
    import torch
    from paper_2608_06412_amd import Context, default_config
    rng = np.random.default_rng(8)
    ctx = Context(default_config(0.01, 0.04, r_c=0.01, max_blocks=1 << 14, max_points=1 << 16,
                                 max_orientations=512, max_tools=3))
    for i, K in enumerate((64, 256, 300)):
        ctx.set_tool_kernels(i, synth_mod.cylinder_tool(0.02, 0.1, 0.3),
                             synth_mod.orientations(synth_mod.fibonacci_directions(K), 1))
    corners = ((0, 0, 0), (60, 0, 0), (0, 60, 0), (60, 60, 0))
    for j in range(4):
        xyz = np.concatenate([patch(rng, c) for c in corners]).astype(np.float32)
        o = np.array([30.0, 30.0, 2.0], np.float32) + np.float32(20) * rng.uniform(-1, 1, 3).astype(np.float32) * [1, 1, 0]
        ctx.integrate_frame(torch.from_numpy(xyz).cuda(), o.astype(np.float32), j)
    best = ctx.score_variant_default()
    want = []
    for i in range(3):
        out = []
        for v in (best, 0):
            ctx.set_score_variant(v)
            ctx.score_points(i)
            lab = ctx.read_labels(i)
            out.append((lab["label"].tolist(), lab["first_free"].tolist(),
                        {k: x for k, x in ctx.score_stats(i).items() if k in (
                            "n_confident", "n_accessible", "n_blocked", "n_no_candidate",
                            "canonical_tests", "canonical_lookups")}))
        assert out[0] == out[1]
        assert out[0][2]["n_accessible"] > 100 and out[0][2]["n_blocked"] > 100, out[0][2]
        want.append(out[0])
    ctx.set_score_variant(best)
    ctx.score_tools([0, 1, 2])
    for i in range(3):
        lab = ctx.read_labels(i)
        assert (lab["label"].tolist(), lab["first_free"].tolist()) == want[i][:2]
