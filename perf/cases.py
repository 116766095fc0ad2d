"""The work a program has this framework do, as measurable cases.

A program streams LiDAR frames into a map (integrate), asks which surface
points a tool can reach (score) and reads the labels; it does so eagerly, as
a recorded frame graph, with a sliding window, incrementally, for several
tools at once or for several sensors on one server, and it refines approach
directions with the differentiable smoothed score.  Each case is one such
call sequence through the public entry points, at a size between the
smallest scene the repository works with (2,000 returns, 2 cm voxels, 64
orientations) and its largest (the tree map of 300 frames of 20,000 returns,
1 cm voxels, 256 orientations; eight tools of 512 orientations).

Scenes are seeded and made here: a tree of tapered limbs, a cluster of boxes
on a slab, a sphere beside a box.  A frame is what a spinning sensor would
return from a pose: surface samples facing the sensor, thinned by solid
angle, hidden ones removed by a depth buffer, with Gaussian range noise.
"""
import math

import numpy as np
import torch

from paper_2608_06412_amd import Context, Server, default_config
from paper_2608_06412_amd.smooth import smooth_score

R_C = 0.01       # collision threshold, metres
LAP = 48         # frames a measured state goes round (the sensor's next frames)
C_CLEAR, TAU_S = 0.01, 0.005   # smoothed score: clearance and softness, metres
ETA = 2e-7       # ascent step: under a degree a step, so that the ascent follows its gradient


# --------------------------------------------------------------------------
# scenes and frames
# --------------------------------------------------------------------------
def _tree(rng):
    """Limbs (start, end, radius): an 8 m trunk and four levels of branches."""
    limbs = []
    for i in range(8):
        limbs.append([0, 0, i, 0, 0, i + 1, 0.20 * (1 - 0.75 * (i + 0.5) / 8)])

    def grow(p0, d, length, radius, level):
        p1 = p0 + d * length
        limbs.append([*p0, *p1, radius])
        if level == 5:
            return
        for _ in range(int(rng.integers(3, 6))):
            az, el = rng.uniform(0, 2 * math.pi), math.radians(rng.uniform(20, 70))
            e = np.array([math.cos(el) * math.cos(az), math.cos(el) * math.sin(az), math.sin(el)])
            grow(p0 + (p1 - p0) * rng.uniform(0.3, 0.95), e, length * 0.6 * rng.uniform(0.85, 1.15),
                 radius * 0.5, level + 1)

    for _ in range(4):
        az, el = rng.uniform(0, 2 * math.pi), math.radians(rng.uniform(20, 70))
        e = np.array([math.cos(el) * math.cos(az), math.cos(el) * math.sin(az), math.sin(el)])
        grow(np.array([0, 0, rng.uniform(2, 7.5)]), e, 1.6 * rng.uniform(0.85, 1.15), 0.15, 1)
    return np.array(limbs, np.float64), np.zeros((0, 6)), np.zeros((0, 4))


def _cluster(rng):
    """Boxes (low corner, high corner): twelve of 10-80 cm on a 6 x 6 m slab."""
    boxes = [[-3, -3, -0.2, 3, 3, 0.0]]
    for _ in range(12):
        c, s = rng.uniform(-2.1, 2.1, 2), rng.uniform(0.1, 0.8, 3)
        z = 0.0 if rng.uniform() < 0.7 else rng.uniform(0.2, 1.0)
        boxes.append([c[0] - s[0] / 2, c[1] - s[1] / 2, z, c[0] + s[0] / 2, c[1] + s[1] / 2, z + s[2]])
    return np.zeros((0, 7)), np.array(boxes), np.zeros((0, 4))


def _sphere(rng):
    """A 1 m sphere beside a 40 cm box (moved a little by the seed)."""
    d = rng.uniform(-0.05, 0.05, 2)
    return (np.zeros((0, 7)), np.array([[0.8 + d[0], -0.2 + d[1], 0, 1.2 + d[0], 0.2 + d[1], 0.4]]),
            np.array([[0, 0, 0.5, 0.5]]))


SCENES = {"tree": _tree, "cluster": _cluster, "sphere": _sphere}


def _poses(scene, n):
    """Sensor positions: an orbit of 4-6 m that climbs the tree, or a circle
    above the smaller scenes."""
    t = np.arange(n)
    if scene == "tree":
        a, r = 2 * np.pi * t / 150, 5 + np.sin(2 * np.pi * t / 345)
        return np.stack([r * np.cos(a), r * np.sin(a), 4.25 - 3.75 * np.cos(2 * np.pi * t / 600)], 1)
    a = 2 * np.pi * t / 60
    r, z = (2.6, 1.4) if scene == "cluster" else (3.0, 1.5)
    return np.stack([0.3 + r * np.cos(a), r * np.sin(a), np.full(n, z)], 1)


class _Surface:
    """Area-uniform samples (position, normal) of a scene, on the GPU."""

    def __init__(self, scene, gen):
        self.gen = gen
        limbs, boxes, balls = (torch.from_numpy(np.asarray(a, np.float64)).float().cuda() for a in scene)
        self.limbs, self.boxes, self.balls = limbs, boxes, balls
        d = limbs[:, 3:6] - limbs[:, :3]
        self.len = d.norm(dim=1)
        self.ax = d / self.len[:, None].clamp_min(1e-9)
        up = torch.where(self.ax[:, 2:].abs() < 0.9, torch.tensor([0.0, 0, 1]).cuda(),
                         torch.tensor([1.0, 0, 0]).cuda()) if len(limbs) else d
        self.e1 = torch.linalg.cross(up, self.ax) if len(limbs) else d
        self.e1 = self.e1 / self.e1.norm(dim=1, keepdim=True).clamp_min(1e-9)
        self.e2 = torch.linalg.cross(self.ax, self.e1) if len(limbs) else d
        e = boxes[:, 3:] - boxes[:, :3]
        self.ext = e
        faces = torch.stack([e[:, 1] * e[:, 2], e[:, 0] * e[:, 2], e[:, 0] * e[:, 1]], 1)
        self.faces = faces.repeat_interleave(2, 1).reshape(-1)          # box, axis, side
        self.areas = [2 * math.pi * limbs[:, 6] * self.len, self.faces, 4 * math.pi * balls[:, 3] ** 2]
        tot = [float(a.sum()) for a in self.areas]
        self.share = [t / sum(tot) for t in tot]
        self.cum = [a.cumsum(0) / max(t, 1e-9) for a, t in zip(self.areas, tot)]

    def sample(self, n):
        pos, nrm = [], []
        for kind, share in enumerate(self.share):
            m = int(round(n * share))
            if m == 0:
                continue
            u = torch.rand((m, 3), generator=self.gen, device="cuda")
            i = torch.searchsorted(self.cum[kind], u[:, 0].contiguous()).clamp_max(len(self.cum[kind]) - 1)
            if kind == 0:
                ph = 2 * math.pi * u[:, 1:2]
                v = torch.cos(ph) * self.e1[i] + torch.sin(ph) * self.e2[i]
                p = self.limbs[i, :3] + u[:, 2:] * (self.ax * self.len[:, None])[i] + self.limbs[i, 6:] * v
            elif kind == 1:
                b, ax, side = i // 6, (i % 6) // 2, i % 2
                w = torch.rand((m, 3), generator=self.gen, device="cuda")
                w.scatter_(1, ax[:, None], side[:, None].float())
                p = self.boxes[b, :3] + w * self.ext[b]
                v = torch.zeros_like(w).scatter_(1, ax[:, None], 2 * side[:, None].float() - 1)
            else:
                z, ph = 2 * u[:, 1] - 1, 2 * math.pi * u[:, 2]
                r = (1 - z * z).clamp_min(0).sqrt()
                v = torch.stack([r * torch.cos(ph), r * torch.sin(ph), z], 1)
                p = self.balls[i, :3] + self.balls[i, 3:] * v
            pos.append(p)
            nrm.append(v)
        return torch.cat(pos), torch.cat(nrm)


def _frame(surf, pose, n, sigma):
    """n returns seen from `pose` (float32 [n, 3], on the GPU)."""
    q = torch.tensor(pose, dtype=torch.float32, device="cuda")
    got, have = [], 0
    for _ in range(6):
        p, v = surf.sample(12 * n)
        d = p - q
        r = d.norm(dim=1)
        u = d / r[:, None]
        cos = -(u * v).sum(1)
        az = ((torch.atan2(u[:, 1], u[:, 0]) + math.pi) * (180 / math.pi / 0.4)).long()
        el = ((torch.asin(u[:, 2].clamp(-1, 1)) + math.pi / 2) * (180 / math.pi / 0.4)).long()
        cell = az * 452 + el
        far = torch.where(cos > 0, r, torch.full_like(r, 1e9))
        near = torch.full((902 * 452,), 1e9, device="cuda").scatter_reduce_(0, cell, far, "amin")
        thin = torch.rand(len(r), generator=surf.gen, device="cuda") * r * r < cos * far.min() ** 2 * 4
        keep = (cos > 0.05) & thin & (r < near[cell] + 0.08)
        noise = torch.randn(len(r), generator=surf.gen, device="cuda") * sigma
        x = (p + noise[:, None] * u)[keep]
        got.append(x[torch.randperm(len(x), generator=surf.gen, device="cuda")])
        have += len(x)
        if have >= n:
            break
    x = torch.cat(got)
    return x[torch.arange(n, device="cuda") % len(x)].contiguous()


def _frames(case, seed, n):
    """n frames of the case: [(returns, sensor position, frame id)]."""
    gen = torch.Generator(device="cuda").manual_seed(1000003 * (seed % 100003) + 17)
    surf = _Surface(SCENES[case["scene"]](np.random.default_rng(seed)), gen)
    poses = _poses(case["scene"], n).astype(np.float32)
    sigma = 0.02 if case["scene"] == "tree" else 0.01
    uneven = np.random.default_rng(seed + 1).uniform(0.25, 1.75, n) if case.get("uneven") else np.ones(n)
    return [(_frame(surf, poses[i], max(1, int(case["returns"] * uneven[i])), sigma), poses[i], i)
            for i in range(n)]


# --------------------------------------------------------------------------
# tools and orientations
# --------------------------------------------------------------------------
def _directions(n):
    k = np.arange(n)
    z = 1 - (2 * k + 1) / n
    r, a = np.sqrt(np.maximum(0, 1 - z * z)), k * math.pi * (3 - math.sqrt(5))
    return np.stack([r * np.cos(a), r * np.sin(a), z], 1)


def _orientations(n_dirs, n_roll):
    """Row-major rotation matrices, n_roll rolls of each of n_dirs directions."""
    out = []
    for d in _directions(n_dirs):
        a = np.array([0.0, 0, 1]) if abs(d[2]) < 0.9 else np.array([1.0, 0, 0])
        e1 = d / np.linalg.norm(d)
        e2 = np.cross(a, e1)
        e2 /= np.linalg.norm(e2)
        e3 = np.cross(e1, e2)
        for k in range(n_roll):
            c, s = math.cos(k * math.pi / n_roll), math.sin(k * math.pi / n_roll)
            out.append(np.stack([e1, c * e2 + s * e3, c * e3 - s * e2], 1).reshape(9))
    return np.array(out)


def _tool(i, corridor):
    """Tool 0: the 30 x 5 x 2 cm saw box; others: cylinders (odd) and boxes
    (even) of 2-8 cm cross-section and 10-30 cm length."""
    if i == 0:
        return dict(shape=1, length=0.30, corridor=corridor, r_s=math.hypot(0.025, 0.01), width=0.05, height=0.02)
    rng = np.random.default_rng(13 + i)
    size, length, reach = rng.uniform(0.02, 0.08), rng.uniform(0.10, 0.30), corridor * rng.uniform(0.3, 1.5)
    if i % 2:
        return dict(shape=0, length=length, corridor=reach, r_s=size / 2, radius=size / 2)
    h = rng.uniform(0.02, size)
    return dict(shape=1, length=length, corridor=reach, r_s=math.hypot(size / 2, h / 2), width=size, height=h)


def _samples(tool):
    """The tool solid as 64 points: 16 stations along it, four rim points each."""
    y, z = tool["width"] / 2, tool["height"] / 2
    xs = np.linspace(tool["r_s"], tool["length"] + tool["corridor"], 16)
    return np.array([[x, a, b] for x in xs for a, b in ((y, z), (-y, z), (-y, -z), (y, -z))], np.float32)


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # the smallest scene: every frame integrated, scored and read back at
        # once; latency and launches count
        dict(name="frame_tiny", kind="frame", scene="sphere", returns=2000, before=12, voxel=0.02, dirs=64, rolls=1,
             corridor=0.5),
        # an odd orientation count above 256 and an odd frame, mid-sized map
        dict(name="frame_odd", kind="frame", scene="cluster", returns=7919, before=40, voxel=0.015, dirs=97, rolls=3,
             corridor=0.7),
        # the main loop: a frame of the tree survey integrated and scored
        dict(name="frame_tree", kind="frame", scene="tree", returns=20000, before=150, voxel=0.01, dirs=64, rolls=4,
             corridor=1.0),
        # the same frame replayed as a recorded graph, as a control loop does
        dict(name="graph_tree", kind="graph", scene="tree", returns=20000, before=80, voxel=0.01, dirs=64, rolls=4,
             corridor=1.0),
        # mapping from a driver's host buffers at frame rate, scored now and
        # then: four large frames integrated, one scoring
        dict(name="ingest_host", kind="ingest", scene="cluster", returns=40000, before=20, voxel=0.02, dirs=64,
             rolls=1, corridor=0.5),
        # a finished survey scored for a tool (1.9 M points, 256 orientations)
        dict(name="score_survey", kind="score", scene="tree", returns=20000, before=300, voxel=0.01, dirs=64, rolls=4,
             corridor=1.0),
        # eight tools of 512 orientations on one map, frames of uneven size
        dict(name="tools_batch", kind="tools", scene="tree", returns=22500, before=40, voxel=0.01, dirs=128, rolls=4,
             corridor=1.0, tools=8, uneven=True),
        # the 10 m sliding window following the sensor round the tree
        dict(name="window_tree", kind="window", scene="tree", returns=20000, before=100, voxel=0.01, dirs=64, rolls=4,
             corridor=1.0, window=10.0),
        # the incremental mode: only queued points re-evaluated
        dict(name="incremental_tree", kind="incremental", scene="tree", returns=20000, before=100, voxel=0.01,
             dirs=64, rolls=4, corridor=1.0),
        # four sensors on one server, one frame of each per step
        dict(name="serve_four", kind="serve", scene="tree", returns=22500, before=30, voxel=0.01, dirs=64, rolls=4,
             corridor=0.6, streams=4, uneven=True),
        # one step of a gradient-based planner: score and gradients of 1,000
        # poses, forward and backward
        dict(name="smooth_step", kind="smooth", scene="cluster", returns=8000, before=24, voxel=0.02, pairs=1000,
             corridor=0.5),
        # approach directions of 4,000 points refined from 64 starts each
        dict(name="refine_tree", kind="refine", scene="tree", returns=20000, before=48, voxel=0.01, pairs=4000,
             starts=64, steps=20, corridor=1.0),
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["frame", "frame", "graph", "ingest", "score", "tools", "window", "incremental", "serve",
                       "smooth", "smooth", "refine"])
    scene = rng.choice(["sphere", "cluster", "tree", "tree"])
    voxel = rng.choice([0.01, 0.0125] if scene == "tree" else [0.0125, 0.015, 0.02])
    c = dict(kind=kind, scene=scene, voxel=voxel, corridor=round(rng.uniform(0.3, 1.2), 2),
             returns=log(2000, 20000 if kind in ("serve", "tools") else 40000))
    c["before"] = log(8, 120 if c["returns"] <= 20000 else 60)
    if kind in ("smooth", "refine"):
        c["before"] = min(c["before"], 40)
        c["pairs"] = log(200, 200000) if kind == "smooth" else log(50, 3500)
        if kind == "refine":
            c.update(starts=rng.choice([1, 8, 64]), steps=rng.choice([5, 20]))
        return c
    c["rolls"] = rng.choice([1, 2, 3, 4])
    c["dirs"] = log(24, 512 // c["rolls"] if kind != "tools" else 128)
    if kind == "tools":
        c.update(tools=rng.randint(2, 6), uneven=True)
    elif kind == "window":
        c["window"] = 10.0 if scene == "tree" else 4.0
    elif kind == "serve":
        c.update(streams=rng.randint(2, 4), uneven=True, before=min(c["before"], 40))
    return c


def _pinned(n, dtype):
    return torch.empty(n, dtype=dtype, pin_memory=True).numpy()


def _label_buffers(n):
    """Host arrays for the labels of up to n points, allocated once."""
    out = dict(label=_pinned(n, torch.uint8), first_free=_pinned(n, torch.int16))
    for a in out.values():
        a[:] = 0
    return out


def _capacity(case):
    """Points a state may come to hold: the frames before and one lap."""
    n = int((case["before"] + LAP + 2) * case["returns"] * (1.2 if case.get("uneven") else 1)) + 4096
    return min(n, 1 << 22)


def _config(case, n_points):
    k = case.get("dirs", 1) * case.get("rolls", 1)
    return default_config(case["voxel"], 0.0 if case["voxel"] < 0.02 else 0.06, r_c=R_C, max_blocks=1 << 16,
                          max_points=n_points, max_orientations=max(64, k), max_tools=case.get("tools", 1))


def _box(frames):
    lo = torch.stack([f[0].amin(0) for f in frames]).amin(0).cpu().numpy() - 1
    hi = torch.stack([f[0].amax(0) for f in frames]).amax(0).cpu().numpy() + 1
    return lo, hi


def _step(s):
    """The state's next frame; frame ids go on increasing."""
    f = s["lap"][s["at"] % len(s["lap"])]
    s["at"] += 1
    return f[0], f[1], s["first"] + s["at"]


def _smooth_inputs(case, seed, frames):
    """Points on the surface (voxel centres, in Morton order of their 8^3
    blocks as a planner walks its map), quaternions, samples."""
    gen = torch.Generator(device="cuda").manual_seed(seed + 5)
    allx = torch.cat([f[0] for f in frames])
    x = allx[torch.randint(len(allx), (case["pairs"],), generator=gen, device="cuda")].double()
    vox = torch.floor(x / case["voxel"]).long()
    b = (vox >> 3) - (vox >> 3).amin(0)
    code = torch.zeros(len(b), dtype=torch.int64, device="cuda")
    for bit in range(12):
        for a in range(3):
            code |= ((b[:, a] >> bit) & 1) << (3 * bit + a)
    p = ((vox[torch.argsort(code, stable=True)].double() + 0.5) * case["voxel"]).float()
    smp = torch.from_numpy(_samples(_tool(0, case["corridor"]))).cuda()
    if case["kind"] == "smooth":
        jit = torch.rand((len(p), 3), generator=gen, device="cuda") - 0.5
        q = torch.randn((len(p), 4), generator=gen, device="cuda")
        g = torch.rand(len(p), generator=gen, device="cuda") + 0.5
        return (p + 0.6 * case["voxel"] * jit).contiguous(), q.contiguous(), smp, g
    d = _directions(case["starts"])
    q = np.stack([1 + d[:, 0], 0 * d[:, 0], -d[:, 2], d[:, 1]], 1)
    q = torch.from_numpy(q / np.linalg.norm(q, axis=1, keepdims=True)).float().cuda()
    return p.contiguous(), q.repeat(len(p), 1).contiguous(), smp, None


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return _prepare_serve(case, seed)
    static = kind in ("smooth", "refine", "score")
    frames = _frames(case, seed, case["before"] + (0 if static else LAP))
    cap = _capacity(case)
    ctx = Context(_config(case, cap))
    s = dict(kind=kind, ctx=ctx, at=0, first=case["before"], lap=frames[case["before"]:])
    if kind in ("smooth", "refine"):
        for x, o, i in frames:
            ctx.integrate_frame(x, o, i)
        s["p"], s["q"], s["samples"], s["g"] = _smooth_inputs(case, seed, frames)
        s["steps"] = case.get("steps")
        if kind == "smooth":
            s["p"].requires_grad_()
            s["q"].requires_grad_()
        return s
    rot = _orientations(case["dirs"], case["rolls"])
    n_tools = case.get("tools", 1)
    small = case["scene"] != "tree"
    for i in range(n_tools):
        tool = dict(shape=0, length=0.10, corridor=case["corridor"], r_s=0.03, radius=0.03) if small and n_tools == 1 \
            else _tool(i, case["corridor"])
        ctx.set_tool_kernels(i, tool, rot)
    if kind == "window":
        ctx.set_window([max(2, math.ceil(case["window"] / (8 * case["voxel"])))] * 3)
    if kind == "incremental":
        ctx.incremental_enable(0, 1 << 20)
    early = frames[:case["before"]]
    if kind == "graph":
        lo, hi = _box(frames)
        ctx.graph_prepare(lo, hi, max(len(f[0]) for f in frames), [0])
        for x, o, i in early:
            ctx.graph_frame(x, o, i)
        ctx.graph_sync()
    else:
        for x, o, i in early:
            (ctx.incremental_frame if kind == "incremental" else ctx.integrate_frame)(x, o, i)
    s["tools"] = list(range(n_tools))
    s["out"] = [_label_buffers(cap) for _ in range(n_tools)]
    if kind == "ingest":   # a driver hands over ordinary host arrays
        s["lap"] = [(x.cpu().numpy(), o, i) for x, o, i in s["lap"]]
    return s


def _prepare_serve(case, seed):
    srv = Server(64 << 30, max_streams=case["streams"])
    s = dict(kind="serve", srv=srv, sids=[], lap=[], at=0, first=case["before"], out=[])
    rot = _orientations(case["dirs"], case["rolls"])
    for k in range(case["streams"]):
        mine = dict(case, scene=case["scene"] if k % 2 == 0 else "cluster")
        frames = _frames(mine, seed + 101 * k, case["before"] + LAP)
        cap = _capacity(case)
        cfg = _config(case, cap)
        cfg.hbm_budget = 8 << 30
        sid = srv.admit(cfg)
        ctx = srv.context(sid)
        ctx.set_tool_kernels(0, _tool(k, case["corridor"]), rot)
        lo, hi = _box(frames)
        srv.prepare(sid, lo, hi, max(len(f[0]) for f in frames), [0])
        for x, o, i in frames[:case["before"]]:
            ctx.graph_frame(x, o, i)
        ctx.graph_sync()
        s["sids"].append(sid)
        s["lap"].append([(x.cpu().numpy(), o) for x, o, _ in frames[case["before"]:]])
        s["out"].append(_label_buffers(cap))
    return s


def run(s):
    kind = s["kind"]
    if kind == "smooth":
        v = smooth_score(s["ctx"], s["p"], s["q"], s["samples"], C_CLEAR, TAU_S)
        dp, dq = torch.autograd.grad(v, (s["p"], s["q"]), s["g"])
        return dict(s=v.detach(), dp=dp, dq=dq)
    if kind == "refine":
        q, v = s["ctx"].smooth_refine(s["p"], s["q"], s["samples"], steps=s["steps"], eta=ETA, max_step=0.05,
                                      c=C_CLEAR, tau_s=TAU_S)
        return dict(q=q, s=v)
    if kind == "serve":
        fid = s["first"] + s["at"] + 1
        for k, sid in enumerate(s["sids"]):
            x, o = s["lap"][k][s["at"] % len(s["lap"][k])]
            s["srv"].submit(sid, x, o, fid)
        s["at"] += 1
        for sid, _, status in s["srv"].step():
            if status != 0:
                raise RuntimeError("stream %d: %s" % (sid, s["srv"].last_error()))
        for sid, out in zip(s["sids"], s["out"]):
            s["srv"].context(sid).read_labels(0, out=out, keys=False)
        return s["out"]
    ctx = s["ctx"]
    if kind == "incremental":
        ctx.incremental_frame(*_step(s))
        ctx.read_incremental(labels_only=True, label_out=s["out"][0]["label"], keys=False)
        return s["out"][0]["label"]
    if kind == "graph":
        ctx.graph_frame(*_step(s))
        ctx.graph_sync()
    elif kind == "score":
        ctx.score_points(0)
    else:
        for _ in range(4 if kind == "ingest" else 1):
            ctx.integrate_frame(*_step(s))
        if kind == "tools":
            ctx.score_tools(s["tools"])
        else:
            ctx.score_points(0)
    for t in s["tools"]:
        ctx.read_labels(t, out=s["out"][t], keys=False)
    return s["out"]


def _points(case):
    """About how many surface points the map holds: noisy returns fill the
    voxels near the surface, fewer new ones each frame."""
    area, sigma = {"tree": (45.0, 0.02), "cluster": (60.0, 0.01), "sphere": (3.5, 0.01)}[case["scene"]]
    room = area / case["voxel"] ** 2 * (1 + 4 * sigma / case["voxel"])
    return room * (1 - math.exp(-case["returns"] * (case["before"] + LAP / 2) / room))


def work(case):
    """Bytes: each return (12), each point's key, weight, sensor sum, normal
    and stored viewpoints (160) read, its label and orientation (3) written;
    each smoothed pair's pose, score and gradients.  Operations: one test of
    six table entries per point and orientation (a sixth of the sensor side's
    orientations get that far), 40 per smoothed sample and evaluation, 20 per
    return and voxel of its cube."""
    if case["kind"] in ("smooth", "refine"):
        n = case["pairs"] * case.get("starts", 1)
        evals = case["steps"] + 1 if case["kind"] == "refine" else 2
        return {"bytes": 48 * n + 64 * 12, "flops": 40.0 * 64 * n * evals}
    sets = case.get("tools", 1)
    n = _points(case) * case.get("streams", 1)
    frames = {"ingest": 4, "score": 0}.get(case["kind"], 1) * case.get("streams", 1)
    seen = 0.35 if case["kind"] in ("incremental", "window") else 1.0
    r = math.ceil(min(4 * case["voxel"], 0.1) / case["voxel"] - 1e-9) if case["voxel"] < 0.02 else 3
    cube = (2 * r + 1) ** 3
    return {"bytes": frames * case["returns"] * (12.0 + 6 * cube / 8) + n * (160.0 * seen + 3 * sets),
            "flops": frames * case["returns"] * cube * 20.0 + 6.0 * n * seen * sets * case["dirs"] * case["rolls"]}


# --------------------------------------------------------------------------
# the smoothed score in 64 bits
# --------------------------------------------------------------------------
def _isqrt(n):
    r = torch.sqrt(n.double()).long()
    r = torch.where(r * r > n, r - 1, r)
    return torch.where((r + 1) * (r + 1) <= n, r + 1, r)


def _field(case, frames):
    """The signed distance of every voxel (metres, truncation where nothing
    was seen) as the definition of the map gives it, on a dense grid."""
    v = case["voxel"]
    scale, tau = 256.0 / v, 0.06 if v >= 0.02 else min(4 * v, 0.1)
    tau_u = int(round(tau * scale))
    R = (tau_u + 255) // 256
    P = [torch.round(f[0].double() * scale).long() for f in frames]
    lo = torch.stack([p.amin(0) for p in P]).amin(0).div(256, rounding_mode="floor") - R - 2
    hi = torch.stack([p.amax(0) for p in P]).amax(0).div(256, rounding_mode="floor") + R + 3
    dim = (hi - lo).tolist()
    S = torch.zeros(dim[0] * dim[1] * dim[2], dtype=torch.int64, device="cuda")
    W = torch.zeros(len(S), dtype=torch.int32, device="cuda")
    k = torch.arange(-R, R + 1, device="cuda")
    cube = torch.stack(torch.meshgrid(k, k, k, indexing="ij"), -1).reshape(-1, 3)
    for (_, o, _), p_all in zip(frames, P):
        Q = torch.from_numpy(np.rint(o.astype(np.float64) * scale).astype(np.int64)).cuda()
        idx, dist = [], []
        for p in p_all.split(8192):
            b = p - Q
            vox = p.div(256, rounding_mode="floor")[:, None] + cube
            a = 256 * vox + 128 - p[:, None]
            ab = (a * b[:, None]).sum(-1).double()
            aa, bb = (a * a).sum(-1).double(), (b * b).sum(-1).double()
            use = ~((ab > 0) & (400 * ab * ab > 361 * aa * bb[:, None]))
            c = 256 * vox + 128 - Q
            d = _isqrt((b * b).sum(-1))[:, None] - _isqrt((c * c).sum(-1))
            vox = vox - lo
            lin = (vox[..., 0] * dim[1] + vox[..., 1]) * dim[2] + vox[..., 2]
            idx.append(lin[use])
            dist.append(d[use].clamp(0, tau_u))
        idx, dist = torch.cat(idx), torch.cat(dist)
        S.index_add_(0, idx, dist)
        W.index_add_(0, idx, torch.ones_like(idx, dtype=torch.int32))
        if int(W.max()) > 2000:
            over = W > 2000
            S[over] = (S[over] * 2000).div(W[over].long(), rounding_mode="floor")
            W[over] = 2000
    T = torch.where(W > 0, S.double() / W.clamp_min(1) / scale, torch.full_like(S, 0, dtype=torch.float64) + tau)
    return T, lo, dim, tau


def _score64(case, field, p, q, smp, grads):
    """s of the pairs in float64 and, with grads, ds/dp and ds/dq."""
    T, lo, dim, tau = field
    p = p.double().detach()
    qn = q.norm(dim=1, keepdim=True)
    w, x, y, z = (q / qn).unbind(1)
    R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    u = torch.matmul(smp.double()[None].expand(len(p), -1, -1), R.transpose(1, 2).contiguous())
    g = (p[:, None] + u) / case["voxel"] - 0.5
    base = torch.floor(g)
    f = g - base
    base = base.long() - lo
    t = []
    for k in range(8):
        c = base + torch.tensor([k & 1, (k >> 1) & 1, k >> 2], device="cuda")
        ok = ((c >= 0) & (c < torch.tensor(dim, device="cuda"))).all(-1)
        lin = (c[..., 0] * dim[1] + c[..., 1]) * dim[2] + c[..., 2]
        t.append(torch.where(ok, T[torch.where(ok, lin, 0)], tau))
    fx, fy, fz = f.unbind(-1)
    a00, a10 = t[0] + fx * (t[1] - t[0]), t[2] + fx * (t[3] - t[2])
    a01, a11 = t[4] + fx * (t[5] - t[4]), t[6] + fx * (t[7] - t[6])
    b0, b1 = a00 + fy * (a10 - a00), a01 + fy * (a11 - a01)
    zz = (b0 + fz * (b1 - b0) - C_CLEAR) / TAU_S
    s = torch.nn.functional.logsigmoid(zz).sum(1)
    if not grads:
        return s
    gx = (1 - fz) * ((1 - fy) * (t[1] - t[0]) + fy * (t[3] - t[2])) + fz * ((1 - fy) * (t[5] - t[4]) + fy * (t[7] - t[6]))
    gy = (1 - fz) * (a10 - a00) + fz * (a11 - a01)
    G = torch.stack([gx, gy, b1 - b0], -1) * (torch.sigmoid(-zz) / TAU_S / case["voxel"])[..., None]
    tq = torch.linalg.cross(u, G).sum(1)
    vec = torch.stack([x, y, z], 1)
    dq = 2 * torch.cat([-(tq * vec).sum(1, keepdim=True), w[:, None] * tq + torch.linalg.cross(tq, vec)], 1) / qn
    return s, G.sum(1), dq


def exact(case, seed):
    if case["kind"] not in ("smooth", "refine"):
        return None   # labels and orientations: whole numbers
    frames = _frames(case, seed, case["before"])
    field = _field(case, frames)
    p, q, smp, g = _smooth_inputs(case, seed, frames)
    out = []
    for at in range(0, len(q), 32768):
        if case["kind"] == "smooth":
            s, dp, dq = _score64(case, field, p[at:at + 32768], q[at:at + 32768].double(), smp, True)
            w = g[at:at + 32768, None].double()
            out.append((s, dp * w, dq * w))
            continue
        qs = q[at:at + 32768].double()
        ps = p[torch.arange(at, at + len(qs), device="cuda") // case["starts"]]
        for _ in range(case["steps"]):
            D = ETA * _score64(case, field, ps, qs, smp, True)[2]
            n = D.norm(dim=1, keepdim=True)
            qs = qs + D * torch.where(n > 0.05, 0.05 / n, torch.ones_like(n))
            qs = qs / qs.norm(dim=1, keepdim=True)
        out.append((qs, _score64(case, field, ps, qs, smp, False)))
    keys = ("s", "dp", "dq") if case["kind"] == "smooth" else ("q", "s")
    return {k: torch.cat([o[i] for o in out]) for i, k in enumerate(keys)}
