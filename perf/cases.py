"""Performance cases of the rendering path: what a simulator, a trainer and an
avatar pipeline call, from one 128 x 128 preview to sixteen 640 x 480 avatar
views with their gradients.

listed() names the cases and says what each stands for, draw() gives more of
the same ranges, prepare() makes a case's inputs from a seed, run() is one pass
through the public entry points, work() counts what such a pass cannot do
without and exact() gives its outputs in 64 bits (plain torch, no kernel of
this repository).
"""
import math

import torch

from paper_2604_12626_amd import binding as B
from paper_2604_12626_amd import render
from paper_2604_12626_amd import synth

DEV = "cuda"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _frame(name, n, degree, width, height, views=1, scenes=1, mode="graph", room=True, avatars=0, per_avatar=0):
    return {"name": name, "kind": "frame", "mode": mode, "room": room, "n": n, "degree": degree, "width": width,
            "height": height, "views": views, "scenes": scenes, "avatars": avatars, "per_avatar": per_avatar}


def _train(name, n, degree, width, height, views=1, mode="autograd", depth_loss=False, avatars=0, per_avatar=0):
    return {"name": name, "kind": "train", "mode": mode, "room": True, "n": n, "degree": degree, "width": width,
            "height": height, "views": views, "scenes": 1, "depth_loss": depth_loss, "avatars": avatars,
            "per_avatar": per_avatar}


def listed():
    return [
        # an asset preview: few Gaussians, a small image, called eagerly -- latency and launches
        _frame("preview_eager", 10_000, 0, 128, 128, mode="eager", room=False),
        # odd sizes called eagerly: three small cameras of a small room, partial tiles on both axes
        _frame("odd_views_eager", 120_001, 1, 333, 217, views=3, mode="eager"),
        # one agent's camera in a captured room, replayed every simulator step
        _frame("agent_frame", 1_000_000, 3, 640, 480),
        # a vectorised simulator: 64 agents in 8 scenes of very different sizes, one launch sequence
        _frame("agents_batch", 2_000_000, 3, 256, 256, views=64, scenes=8),
        # 16 views of a room with 8 walking avatars, skinned in the same graph
        _frame("avatar_views", 1_000_000, 3, 640, 480, views=16, avatars=8, per_avatar=50_000),
        # a full-HD recording of a large capture
        _frame("hd_frame", 2_000_000, 3, 1920, 1080),
        # scene optimisation: one autograd step on one training view
        _train("train_view", 500_000, 3, 256, 256),
        # scene optimisation at capture resolution, with a depth term
        _train("train_hd_depth", 1_000_000, 3, 1280, 720, depth_loss=True),
        # joint optimisation of a room and its avatars through the skinning, replayed as one graph
        _train("train_avatars", 1_000_000, 3, 640, 480, views=16, mode="graph", avatars=8, per_avatar=50_000),
        # pose fitting: skinning, its canonical gradients and its joint-matrix gradients
        {"name": "pose_fit", "kind": "skin", "avatars": 8, "per_avatar": 50_000},
        # the observation hand-off of 16 agents against a mesh pass
        {"name": "sensor_mesh", "kind": "sensor", "views": 16, "width": 640, "height": 480, "mesh": True},
        # navigation queries of a large crowd of agents against walking avatars
        {"name": "capsules", "kind": "capsules", "agents": 4096, "avatars": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "batch", "avatars", "train", "train", "train_avatars", "skin",
                       "sensor", "capsules"))
    w, h = _log(rng, 96, 1400), _log(rng, 80, 900)
    if kind == "frame":
        c = _frame("", _log(rng, 10_000, 1_500_000), rng.randint(0, 3), w, h,
                   views=rng.choice((1, 1, 2, 3)) if w * h < 300_000 else 1, mode=rng.choice(("graph", "eager")),
                   room=rng.random() < 0.8)
        if not c["room"]:
            c["n"] = min(c["n"], 60_000)
    elif kind == "batch":
        c = _frame("", _log(rng, 100_000, 1_500_000), 3, _log(rng, 128, 300), _log(rng, 128, 300),
                   views=rng.randint(8, 48), scenes=rng.randint(2, 8))
    elif kind == "avatars":
        c = _frame("", _log(rng, 100_000, 900_000), rng.randint(1, 3), _log(rng, 200, 640), _log(rng, 150, 480),
                   views=rng.randint(2, 12), avatars=rng.randint(1, 8), per_avatar=_log(rng, 5_000, 50_000))
    elif kind == "train":
        c = _train("", _log(rng, 50_000, 900_000), rng.randint(0, 3), _log(rng, 96, 1000), _log(rng, 96, 700),
                   views=rng.choice((1, 1, 2)), depth_loss=rng.random() < 0.5)
    elif kind == "train_avatars":
        c = _train("", _log(rng, 50_000, 600_000), rng.randint(1, 3), _log(rng, 160, 500), _log(rng, 120, 400),
                   views=rng.randint(1, 8), mode="graph", avatars=rng.randint(1, 6),
                   per_avatar=_log(rng, 5_000, 50_000))
    elif kind == "skin":
        c = {"kind": "skin", "avatars": rng.randint(1, 16), "per_avatar": _log(rng, 2_000, 50_000) + 1}
    elif kind == "sensor":
        c = {"kind": "sensor", "views": rng.randint(1, 16), "width": w, "height": h, "mesh": rng.random() < 0.6}
    else:
        c = {"kind": "capsules", "agents": _log(rng, 16, 16_384), "avatars": rng.randint(1, 16)}
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
class _Draws:
    """Seeded draws on the GPU (or the CPU, for a few numbers)."""

    def __init__(self, seed, device=DEV):
        self.g = torch.Generator(device=device).manual_seed(int(seed) * 7919 + 17)
        self.device = device

    def u(self, *shape):
        return torch.rand(shape, generator=self.g, device=self.device)

    def n(self, *shape):
        return torch.randn(shape, generator=self.g, device=self.device)

    def i(self, hi, *shape):
        return torch.randint(0, hi, shape, generator=self.g, device=self.device)


def _attributes(d, n, degree, mu, sigma):
    q = d.n(n, 4)
    sh = 0.05 * d.n(n, (degree + 1) ** 2, 3)
    sh[:, 0] *= 6.0
    return {"log_scales": mu + sigma * d.n(n, 3), "quats": q / q.norm(dim=1, keepdim=True),
            "opacity": torch.sigmoid(d.n(n)), "sh": sh, "sh_degree": degree}


def _room(d, n, degree):
    """A captured room: 70% of the Gaussians within 5 cm of the floor and walls."""
    size = torch.tensor(synth.ROOM, device=d.device)
    means = d.u(n, 3) * size
    L, W, H = synth.ROOM
    area = torch.tensor([L * W, L * H, L * H, W * H, W * H], device=d.device)
    face = torch.searchsorted(torch.cumsum(area / area.sum(), 0), d.u(n)).clamp(max=4)
    off = 0.05 * d.u(n)
    face = torch.where(d.u(n) < 0.7, face, torch.full_like(face, 5))
    for f, axis, far in ((0, 2, 0.0), (1, 1, 0.0), (2, 1, W), (3, 0, 0.0), (4, 0, L)):
        on = face == f
        means[:, axis] = torch.where(on, far - off if far else off, means[:, axis])
    return {"means": means.contiguous(), **_attributes(d, n, degree, -4.5, 0.7)}


def _cube(d, n, degree):
    means = 2.0 * d.u(n, 3) - 1.0
    means[:, 2] += 3.0
    return {"means": means, **_attributes(d, n, degree, -4.0, 0.5)}


def _cameras(seed, views, width, height, room):
    if not room:
        cams = [synth.identity_camera(float(width), float(width), width / 2.0, height / 2.0) for _ in range(views)]
    else:
        d = _Draws(seed + 555, "cpu")
        cams = []
        for _ in range(views):
            x = d.u(5).tolist()
            pos = [0.5 + x[k] * (synth.ROOM[k] - 1.0) for k in range(3)]
            cams.append(synth.look_camera(pos, 2 * math.pi * x[3], math.radians(40.0 * x[4] - 20.0), width / 2.0,
                                          width / 2.0, width / 2.0, height / 2.0))
    return torch.stack([torch.from_numpy(c) for c in cams]).to(DEV)


def _joint_matrices(seed, count):
    """Joint matrices [count, 24, 12] of random poses of the synthetic
    skeleton, standing somewhere in the room (forward kinematics in 64 bits)."""
    d = _Draws(seed + 777, "cpu")
    w = 0.3 * d.n(count, synth.N_JOINTS, 3).double()
    th = w.norm(dim=-1)[..., None, None].clamp_min(1e-9)
    Z = torch.zeros(count, synth.N_JOINTS, dtype=torch.float64)
    X = torch.stack([Z, -w[..., 2], w[..., 1], w[..., 2], Z, -w[..., 0], -w[..., 1], w[..., 0], Z], -1)
    X = X.view(count, synth.N_JOINTS, 3, 3)
    rot = torch.eye(3, dtype=torch.float64) + torch.sin(th) / th * X + (1 - torch.cos(th)) / th ** 2 * (X @ X)
    yaw = 2 * math.pi * d.u(count).double()
    c, s, z, o = torch.cos(yaw), torch.sin(yaw), torch.zeros(count).double(), torch.ones(count).double()
    parent_R = torch.stack([c, -s, z, s, c, z, z, z, o], -1).view(count, 3, 3)
    parent_t = torch.stack([1.0 + d.u(count).double() * (synth.ROOM[0] - 2), 1.0 + d.u(count).double() *
                            (synth.ROOM[1] - 2), z], -1)
    rest = torch.from_numpy(synth.REST)
    R, t, out = [], [], []
    for k in range(synth.N_JOINTS):
        p = int(synth.PARENTS[k])
        Rp, tp = (parent_R, parent_t) if p < 0 else (R[p], t[p])
        step = rest[k] - (rest[p] if p >= 0 else 0.0)
        t.append(tp + Rp @ step)
        R.append(Rp @ rot[:, k])
        out.append(torch.cat([R[k], (t[k] - R[k] @ rest[k])[..., None]], -1).reshape(count, 12))
    return torch.stack(out, 1).float().to(DEV)


def _avatars(seed, avatars, per, degree):
    """Canonical Gaussians along the bones of the skeleton, four joints each."""
    d = _Draws(seed + 333)
    n = avatars * per
    kids = torch.tensor([k for k in range(synth.N_JOINTS) if synth.PARENTS[k] >= 0], device=DEV)
    rest = torch.from_numpy(synth.REST).float().to(DEV)
    par = torch.from_numpy(synth.PARENTS).to(DEV)
    k = kids[d.i(len(kids), n)]
    t, off = d.u(n, 1), d.n(n, 3)
    off = 0.06 * off / off.norm(dim=1, keepdim=True) * d.u(n, 1) ** (1 / 3)
    w = -torch.log(d.u(n, 4).clamp_min(1e-6))
    g = {"means": rest[par[k]] * (1 - t) + rest[k] * t + off, **_attributes(d, n, degree, -5.0, 0.5)}
    return {**g, "joint_idx": d.u(n, synth.N_JOINTS).topk(4, dim=1).indices.to(torch.uint8).contiguous(),
            "weights": w / w.sum(1, keepdim=True),
            "avatar_of": torch.arange(avatars, device=DEV, dtype=torch.int32).repeat_interleave(per)}


def _target(seed, views, width, height):
    d = _Draws(seed + 999)
    coarse = d.u(views, 3, max(2, height // 32), max(2, width // 32))
    up = torch.nn.functional.interpolate(coarse, size=(height, width), mode="bilinear", align_corners=False)
    return up.permute(0, 2, 3, 1).contiguous()


def _scene(case, seed):
    """Segments, cameras, view -> segment lists and avatar assets of a case."""
    d = _Draws(seed)
    S = case["scenes"]
    # scenes of one batch span a factor of twenty in size
    counts = [max(1, int(case["n"] * 20.0 ** (-s / max(1, S - 1)))) for s in range(S)]
    segs = [(_room if case["room"] else _cube)(d, n, case["degree"]) for n in counts]
    cams = _cameras(seed, case["views"], case["width"], case["height"], case["room"])
    view_segs = [[v % S] for v in range(case["views"])]
    av = None
    if case["avatars"]:
        av = _avatars(seed, case["avatars"], case["per_avatar"], case["degree"])
        if case["kind"] == "frame":  # walking clips of 30 frames, sampled between two of them
            av["clip"] = _joint_matrices(seed, 30 * case["avatars"])
            av["first"] = 30 * torch.arange(case["avatars"], device=DEV, dtype=torch.int32)
            av["frames"] = torch.full((case["avatars"],), 30, device=DEV, dtype=torch.int32)
            av["pos"] = 29.0 * _Draws(seed + 11).u(case["avatars"])
        else:
            av["skin"] = _joint_matrices(seed, case["avatars"])
        view_segs = [v + [S] for v in view_segs]
    return segs, cams, view_segs, av


def _lbs_args(av):
    return av["means"], av["log_scales"], av["quats"], av["joint_idx"], av["weights"], av["avatar_of"]


BG = (0.1, 0.2, 0.3)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sensor":
        return _sensor_inputs(case, seed)
    if kind == "capsules":
        return _capsule_inputs(case, seed)
    if kind == "skin":
        av = _avatars(seed, case["avatars"], case["per_avatar"], 0)
        n, d = case["avatars"] * case["per_avatar"], _Draws(seed + 1)
        e = lambda *s: torch.empty(s, device=DEV)
        return {"kind": kind, "args": _lbs_args(av) + (_joint_matrices(seed, case["avatars"]),),
                "d_out": (d.n(n, 3), d.n(n, 6)), "out": (e(n, 3), e(n, 6)),
                "grads": (e(n, 3), e(n, 3), e(n, 4)), "d_skin": e(case["avatars"], synth.N_JOINTS, 12)}
    segs, cams, view_segs, av = _scene(case, seed)
    # training records checkpoints where the renderer's own rule says they pay
    r = render.Renderer(case["width"], case["height"], bg=BG, checkpoints="auto" if kind == "train" else False)
    state = {"kind": kind, "mode": case["mode"], "renderer": r, "cams": cams, "view_segs": view_segs}
    if kind == "train":
        state["target"] = _target(seed, case["views"], case["width"], case["height"])
        state["depth_loss"] = case["depth_loss"]
    if kind == "train" and case["mode"] == "autograd":
        g = segs[0]
        state["leaves"] = [g[k].requires_grad_(True) for k in ("means", "log_scales", "quats", "opacity", "sh")]
        return state
    before = None
    if av is not None:
        n = av["means"].shape[0]
        posed = {"means": torch.empty(n, 3, device=DEV), "cov6": torch.empty(n, 6, device=DEV),
                 "opacity": av["opacity"], "sh": av["sh"], "sh_degree": av["sh_degree"]}
        segs = segs + [posed]
        if "clip" in av:
            before = lambda: B.deform_lbs_clip(*_lbs_args(av), av["clip"], av["first"], av["frames"], av["pos"],
                                               posed["means"], posed["cov6"])
        else:
            before = lambda: B.deform_lbs(*_lbs_args(av), av["skin"], posed["means"], posed["cov6"])
    state["segs"] = segs
    if case["mode"] == "eager":
        return state
    after = None
    if kind == "train":
        target = state["target"]
        lbs_grads = None if av is None else tuple(torch.empty_like(av[k]) for k in ("means", "log_scales", "quats"))

        def after(f):
            d_rgb = (f.rgb - target) * (2.0 / target.numel())
            grads = r.backward(segs, cams, view_segs, f, d_rgb, None, None)
            if av is not None:
                B.deform_lbs_backward(*_lbs_args(av), av["skin"], grads[-1]["means"], grads[-1]["cov6"], *lbs_grads)
            return grads, lbs_grads

    state["graph"] = render.CapturedRender(r, segs, cams, view_segs, checkpoints=r.checkpoints, before=before,
                                           after=after)
    return state


def _sensor_inputs(case, seed):
    d = _Draws(seed)
    shp = (case["views"], case["height"], case["width"])
    alpha = torch.where(d.u(*shp) < 0.15, torch.zeros(shp, device=DEV), d.u(*shp).clamp_min(1e-4))
    s = {"kind": "sensor", "rgb": 1.2 * d.u(*shp, 3) - 0.1, "alpha": alpha, "depth": alpha * (0.3 + 9.7 * d.u(*shp)),
         "mesh_rgba": None, "mesh_depth": None,
         "out": (torch.empty(shp + (4,), dtype=torch.uint8, device=DEV), torch.empty(shp, device=DEV))}
    if case["mesh"]:
        s["mesh_rgba"] = d.i(256, *shp, 4).to(torch.uint8)
        s["mesh_depth"] = torch.where(d.u(*shp) < 0.15, torch.zeros(shp, device=DEV), 0.3 + 9.7 * d.u(*shp))
    return s


def _capsule_inputs(case, seed):
    """One capsule per bone in clips of 30 frames; agents around the avatars,
    each with a 25 cm step; every agent asks about all avatars."""
    A, E, J = case["avatars"], case["agents"], synth.N_JOINTS
    d = _Draws(seed)
    M = _joint_matrices(seed, A)[:, None].expand(A, 30, J, 12).reshape(A * 30, J, 3, 4).clone()
    walk = (torch.arange(30, device=DEV) * 0.04).repeat(A)
    M[..., 0, 3] += walk[:, None]  # 1.2 m/s at 30 frames a second
    rest = torch.from_numpy(synth.REST).float().to(DEV)
    joints = (M[..., :3] * rest[None, :, None, :]).sum(-1) + M[..., 3]
    kids = [k for k in range(J) if synth.PARENTS[k] >= 0]
    caps = torch.zeros(A * 30, len(kids), 8, device=DEV)
    for c, k in enumerate(kids):
        p = int(synth.PARENTS[k])
        caps[:, c, 0:3], caps[:, c, 4:7] = joints[:, p], joints[:, k]
        caps[:, c, 3] = 0.05 + 0.1 * float((rest[k] - rest[p]).norm())
    who = d.i(A, E)
    pos = torch.zeros(E, 3, device=DEV)
    pos[:, :2] = caps[30 * who, 0, :2] + 3.0 * d.u(E, 2) - 1.5
    yaw = 2 * math.pi * d.u(E)
    nxt = pos + 0.25 * torch.stack([torch.cos(yaw), torch.sin(yaw), torch.zeros(E, device=DEV)], 1)
    span = torch.tensor([[0, A]], dtype=torch.int32, device=DEV).repeat(E, 1)
    return {"kind": "capsules", "pos": pos, "next": nxt, "span": span, "caps": caps,
            "first": 30 * torch.arange(A, device=DEV, dtype=torch.int32),
            "frames": torch.full((A,), 30, device=DEV, dtype=torch.int32), "at": 29.0 * d.u(A),
            "clearance": torch.empty(E, device=DEV), "nearest": torch.empty(E, dtype=torch.int32, device=DEV),
            "gap": torch.empty(E, device=DEV), "blocked": torch.empty(E, dtype=torch.uint8, device=DEV)}


RADIUS, HEIGHT = 0.1, 1.5  # the agents' capsule


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "sensor":
        rgba, depth = render.observation(s["rgb"], s["depth"], s["alpha"], s["mesh_rgba"], s["mesh_depth"],
                                         out=s["out"])
        return {"rgba": rgba, "depth": depth}
    if kind == "capsules":
        B.capsule_queries(s["pos"], s["next"], s["span"], RADIUS, HEIGHT, s["caps"], s["first"], s["frames"],
                          s["at"], s["clearance"], s["nearest"], s["gap"], s["blocked"])
        return {k: s[k] for k in ("clearance", "nearest", "gap", "blocked")}
    if kind == "skin":
        B.deform_lbs(*s["args"], *s["out"])
        B.deform_lbs_backward(*s["args"], *s["d_out"], *s["grads"])
        B.deform_lbs_backward_joints(*s["args"], *s["d_out"], s["d_skin"])
        return {"means": s["out"][0], "cov6": s["out"][1], "d_means": s["grads"][0], "d_log_scales": s["grads"][1],
                "d_quats": s["grads"][2], "d_skin": s["d_skin"]}
    if s["mode"] == "autograd":
        for p in s["leaves"]:
            p.grad = None
        rgb, depth, alpha = render.rasterize(*s["leaves"], s["cams"], s["renderer"])
        loss = (rgb - s["target"]).square().mean()
        if s["depth_loss"]:
            loss = loss + 0.01 * (depth - 2.0 * alpha).square().mean()
        loss.backward()
        return {"rgb": rgb.detach(), "depth": depth.detach(), "alpha": alpha.detach(),
                "grads": [p.grad for p in s["leaves"]]}
    if s["mode"] == "eager":
        f = s["renderer"].render(s["segs"], s["cams"], s["view_segs"])
        return {"rgb": f.rgb, "depth": f.depth, "alpha": f.alpha}
    f = s["graph"].replay()
    out = {"rgb": f.rgb, "depth": f.depth, "alpha": f.alpha}
    if kind == "train":
        grads, lbs = s["graph"].after_out
        out["grads"] = [grads[0][k] for k in ("means", "log_scales", "quats", "opacity", "sh")]
        if lbs is not None:
            out["avatar"] = [*lbs, grads[1]["opacity"], grads[1]["sh"]]
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Bytes: positions of every Gaussian once, the other attributes of the
    share that a view can see (about 15% of a room, all of a cube; several
    views of one scene see up to all of it), the images, and with training the
    dense gradients.  Operations: 26 flop and one exponential per (pixel,
    Gaussian) pair met before the pixel is opaque (about 500 pairs a pixel in
    a room of a million Gaussians, 325 in one of half a million: the square
    root of the size), 70 more per pair for the gradient."""
    kind = case["kind"]
    if kind == "sensor":
        px = case["views"] * case["width"] * case["height"]
        return {"bytes": px * (28 + (8 if case["mesh"] else 0)), "flops": 10 * px}
    if kind == "capsules":
        pairs = case["agents"] * case["avatars"] * 23
        return {"bytes": 45 * case["agents"] + case["avatars"] * 23 * 64, "flops": 460 * pairs}
    if kind == "skin":
        n = case["avatars"] * case["per_avatar"]
        return {"bytes": n * (64 + 36 + 36 + 40), "flops": n * (90 + 200 + 250)}
    px, S = case["views"] * case["width"] * case["height"], case["scenes"]
    row = 32 + 12 * (case["degree"] + 1) ** 2
    total, views = 0, case["views"] / S
    seen = 1.0 - (1.0 - (0.15 if case["room"] else 0.9)) ** views
    pairs = 0.0
    for s in range(S):
        n = max(1, int(case["n"] * 20.0 ** (-s / max(1, S - 1))))
        total += 12 * n + seen * n * row
        pairs += px / S * (500.0 * math.sqrt(n / 1e6) if case["room"] else 60.0)
    n_av = case["avatars"] * case["per_avatar"]
    total += n_av * (96 + 36 + row) + 20 * px
    flops = 27 * pairs + 25 * case["n"] * seen + 90 * n_av
    if kind == "train":
        total += case["n"] * (12 + row) + n_av * (12 + row) + 12 * px
        flops += 71 * pairs
    return {"bytes": total, "flops": flops}


# --------------------------------------------------------------------------
# the outputs in 64 bits
# --------------------------------------------------------------------------
F = torch.float64
T_MIN, A_MIN, A_MAX = (float(torch.tensor(x, dtype=torch.float32)) for x in (1e-4, 1.0 / 255.0, 0.99))


def _rotation(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                        1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                        1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)


def _covariance(g):
    M = _rotation(g["quats"]) * torch.exp(g["log_scales"])[:, None, :]
    return (M[:, :, None, :] * M[:, None, :, :]).sum(-1)


def _harmonics(D, d):
    x, y, z = d.unbind(1)
    xx, yy, zz = x * x, y * y, z * z
    s = lambda a, b: math.sqrt(a / (b * math.pi))
    Y = [torch.full_like(x, s(1, 4))]
    if D >= 1:
        Y += [-s(3, 4) * y, s(3, 4) * z, -s(3, 4) * x]
    if D >= 2:
        Y += [s(15, 4) * x * y, -s(15, 4) * y * z, s(5, 16) * (2 * zz - xx - yy), -s(15, 4) * x * z,
              s(15, 16) * (xx - yy)]
    if D >= 3:
        Y += [-s(35, 32) * y * (3 * xx - yy), s(105, 4) * x * y * z, -s(21, 32) * y * (4 * zz - xx - yy),
              s(7, 16) * z * (2 * zz - 3 * xx - 3 * yy), -s(21, 32) * x * (4 * zz - xx - yy),
              s(105, 16) * z * (xx - yy), -s(35, 32) * x * (xx - 3 * yy)]
    return torch.stack(Y, 1)


def _project64(g, cam, W, H):
    """[m, 10] rows (u, v, A, B, C, opacity, r, g, b, z) with radii and the
    mask of the drawn; g holds 64-bit tensors (rows of one view)."""
    R, t = cam[:9].view(3, 3), cam[9:12]
    fx, fy, cx, cy = cam[12:].unbind()
    m = g["means"]
    x, y, z = ((m[:, None, :] * R).sum(-1) + t).unbind(1)
    front = z > float(torch.tensor(0.2, dtype=torch.float32))
    z = torch.where(front, z, torch.ones_like(z))
    lx, ly = 1.3 * 0.5 * W / fx, 1.3 * 0.5 * H / fy
    xr, yr = (x / z).clamp(-lx, lx), (y / z).clamp(-ly, ly)
    T0 = (fx / z)[:, None] * R[0] - (fx * xr / z)[:, None] * R[2]
    T1 = (fy / z)[:, None] * R[1] - (fy * yr / z)[:, None] * R[2]
    S0, S1 = (g["cov"] * T0[:, None, :]).sum(-1), (g["cov"] * T1[:, None, :]).sum(-1)
    low = float(torch.tensor(0.3, dtype=torch.float32))
    a, b, c = (S0 * T0).sum(-1) + low, (S0 * T1).sum(-1), (S1 * T1).sum(-1) + low
    det = a * c - b * b
    d = m + (R * t[:, None]).sum(0)
    col = (_harmonics(g["sh_degree"], d / d.norm(dim=1, keepdim=True))[:, :, None] * g["sh"]).sum(1) + 0.5
    rows = torch.stack([fx * x / z + cx, fy * y / z + cy, c / det, -b / det, a / det, g["opacity"],
                        *col.clamp(min=0).unbind(1), z], 1)
    with torch.no_grad():
        mid = 0.5 * (a + c)
        lam = mid + torch.sqrt((0.25 * (a - c) ** 2 + b * b).clamp(min=float(torch.tensor(0.1))))
        rad = torch.ceil(3.0 * torch.sqrt(lam)).clamp(max=2.0 ** 24)
        iu, iv = (torch.floor(rows[:, k].clamp(-2.0 ** 20, 2.0 ** 20)) for k in (0, 1))
        x0, x1 = ((iu - rad) // 16).clamp(min=0), ((iu + rad) // 16 + 1).clamp(max=(W + 15) // 16)
        y0, y1 = ((iv - rad) // 16).clamp(min=0), ((iv + rad) // 16 + 1).clamp(max=(H + 15) // 16)
        ok = front & (det > 0) & (x0 < x1) & (y0 < y1)
    return rows, torch.stack([x0, x1, y0, y1], 1).long(), ok


def _lists(z, rect, TX, TY):
    """Sorted tile lists: (row of every key, first key of every tile)."""
    order = torch.sort(z, stable=True).indices
    r = rect[order]
    w, h = r[:, 1] - r[:, 0], r[:, 3] - r[:, 2]
    cnt = w * h
    who = torch.repeat_interleave(torch.arange(len(order), device=z.device), cnt)
    k = torch.arange(len(who), device=z.device) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
    tile = (r[who, 2] + k // w[who]) * TX + r[who, 0] + k % w[who]
    tile, by = torch.sort(tile.int(), stable=True)
    count = torch.bincount(tile.long(), minlength=TX * TY)
    return order[who[by]], torch.cumsum(count, 0) - count, count


def _composite64(rows, rect, W, H, adjoint=None):
    """(rgb [H,W,3], depth, alpha) of one view; with adjoint(rgb, depth,
    alpha) -> their adjoints also the adjoint of `rows`."""
    TX, TY = (W + 15) // 16, (H + 15) // 16
    who, first, count = _lists(rows[:, 9], rect, TX, TY)
    dev = rows.device
    bg = torch.tensor(BG, dtype=torch.float32).to(dev, F)
    img = torch.zeros(TX * TY, 256, 5, dtype=F, device=dev)
    pix = torch.arange(256, device=dev)
    by_len = torch.argsort(count, descending=True)
    lens = count[by_len].tolist()
    px_all, py_all = (by_len % TX)[:, None] * 16 + pix % 16 + 0.5, (by_len // TX)[:, None] * 16 + pix // 16 + 0.5

    groups, at = [], 0
    while at < len(lens):
        L = max(1, lens[at])
        k = max(1, min(len(lens) - at, 40_000_000 // (256 * L)))
        groups.append((at, at + k, L))
        at += k

    def walk(a, b, L):
        t = by_len[a:b]
        j = torch.arange(L, device=dev)[None, :]
        valid = j < count[t][:, None]
        idx = who[(first[t][:, None] + j).clamp(max=max(0, len(who) - 1))] if len(who) else torch.zeros_like(valid, dtype=torch.long)
        e = rows[idx][:, None]  # [tiles, 1, L, 10]
        dx, dy = px_all[a:b][:, :, None] - e[..., 0], py_all[a:b][:, :, None] - e[..., 1]
        P = (-0.5 * (e[..., 2] * dx * dx + e[..., 4] * dy * dy) - e[..., 3] * dx * dy).clamp(max=0)
        raw = e[..., 5] * torch.exp(P)
        al = raw.clamp(max=A_MAX)
        al = torch.where((al >= A_MIN) & valid[:, None], al, torch.zeros_like(al))
        use = (torch.cumprod(1 - al, -1) >= T_MIN) & (al > 0)
        al = al * use
        T = torch.cumprod(1 - al, -1)
        before = T / (1 - al)
        return t, idx, valid, e, dx, dy, raw, al, use, before, T[..., -1]

    for a, b, L in groups:
        if not len(who):
            break
        t, idx, valid, e, dx, dy, raw, al, use, before, Tf = walk(a, b, L)
        w = al * before
        for ch in range(3):
            img[t, :, ch] = (w * e[..., 6 + ch]).sum(-1)
        img[t, :, 3] = (w * e[..., 9]).sum(-1)
        img[t, :, 4] = 1 - Tf
    img[..., :3] += (1 - img[..., 4:]) * bg
    flat = img.view(TY, TX, 16, 16, 5).permute(0, 2, 1, 3, 4).reshape(TY * 16, TX * 16, 5)[:H, :W]
    out = flat[..., :3].contiguous(), flat[..., 3].contiguous(), flat[..., 4].contiguous()
    if adjoint is None:
        return out, None
    d_img = torch.zeros(TY * 16, TX * 16, 5, dtype=F, device=dev)
    d_img[:H, :W] = torch.cat([x if x.dim() == 3 else x[..., None] for x in adjoint(*out)], -1)
    d_img = d_img.view(TY, 16, TX, 16, 5).permute(0, 2, 1, 3, 4).reshape(TX * TY, 256, 5)
    d_rows = torch.zeros_like(rows)
    for a, b, L in groups:
        if not len(who):
            break
        t, idx, valid, e, dx, dy, raw, al, use, before, Tf = walk(a, b, L)
        g = d_img[t]
        w = al * before
        value = e[..., 9] * g[..., 3:4]
        for ch in range(3):
            value = value + e[..., 6 + ch] * g[..., ch:ch + 1]
        got = w * value
        behind = got.sum(-1, keepdim=True) - torch.cumsum(got, -1)
        end = (Tf * ((g[..., :3] * bg).sum(-1) - g[..., 4]))[..., None]
        d_al = torch.where(use, before * value - (behind + end) / (1 - al), torch.zeros_like(al))
        d_P = torch.where(raw > A_MAX, torch.zeros_like(al), d_al * raw)
        d_e = [(d_P * (e[..., 2] * dx + e[..., 3] * dy)).sum(1), (d_P * (e[..., 3] * dx + e[..., 4] * dy)).sum(1),
               (-0.5 * d_P * dx * dx).sum(1), (-d_P * dx * dy).sum(1), (-0.5 * d_P * dy * dy).sum(1),
               d_P.sum(1) / e[:, 0, :, 5], *((w * g[..., ch:ch + 1]).sum(1) for ch in range(4))]
        d_rows.index_add_(0, idx[valid], torch.stack(d_e, -1)[valid])
    return out, d_rows


def _pose64(av, skin):
    A = (av["weights"][:, :, None] * skin[av["avatar_of"].long()[:, None], av["joint_idx"].long()]).sum(1).view(-1, 3, 4)
    M = A[:, :, :3]
    cov = _covariance(av)
    cov = ((M[:, :, None, :] * cov[:, None, :, :]).sum(-1)[:, :, None, :] * M[:, None, :, :]).sum(-1)
    return (M * av["means"][:, None, :]).sum(-1) + A[:, :, 3], cov


def _to64(g):
    return {k: (v.to(F) if torch.is_tensor(v) and v.is_floating_point() else v) for k, v in g.items()}


SIX = ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))


def _exact_images(case, seed):
    segs, cams, view_segs, av = _scene(case, seed)
    train = case["kind"] == "train"
    W, H = case["width"], case["height"]
    segs, cams = [_to64(g) for g in segs], cams.to(F)
    names = ("means", "log_scales", "quats", "opacity", "sh")
    leaves = [[g[k] for k in names] for g in segs]
    if av is not None:
        av = _to64(av)
        leaves.append([av[k] for k in names])
    if train:
        for p in sum(leaves, []):
            p.requires_grad_(True)
        target = _target(seed, case["views"], W, H).to(F)
    with torch.set_grad_enabled(train):
        full = [dict(g, cov=_covariance(g)) for g in segs]
        if av is not None:
            skin = av.get("skin")
            if "clip" in av:
                f = av["pos"].floor().clamp(0, 28)
                s, i = (av["pos"] - f)[:, None, None], av["first"].long() + f.long()
                skin = (1 - s) * av["clip"][i] + s * av["clip"][i + 1]
            means, cov = _pose64(av, skin)
            full.append({"means": means, "cov": cov, "opacity": av["opacity"], "sh": av["sh"],
                         "sh_degree": av["sh_degree"]})
    # the posed tensors are cut here, so that a view's graph can be dropped
    cut = [{k: (v.detach().requires_grad_(train) if torch.is_tensor(v) else v) for k, v in g.items()
            if k in ("means", "cov", "opacity", "sh", "sh_degree")} for g in full]
    images = []
    for v, drawn in enumerate(view_segs):
        parts, keep = [], []
        for s in drawn:
            with torch.no_grad():
                _, rect, ok = _project64(cut[s], cams[v], W, H)
                sel = ok.nonzero()[:, 0]
            with torch.set_grad_enabled(train):
                g = {k: (x[sel] if torch.is_tensor(x) else x) for k, x in cut[s].items()}
                parts.append(_project64(g, cams[v], W, H)[0])
            keep.append(rect[sel])
        with torch.set_grad_enabled(train):
            rows = torch.cat(parts)

        def adjoint(rgb, depth, alpha):
            px = target.shape[0] * W * H
            d = 0.02 / px * (depth - 2 * alpha) if case["depth_loss"] else torch.zeros_like(depth)
            return (rgb - target[v]) * (2.0 / target.numel()), d, -2 * d

        with torch.no_grad():
            img, d_rows = _composite64(rows.detach(), torch.cat(keep), W, H, adjoint if train else None)
        images.append(img)
        if train:
            rows.backward(d_rows)
    out = {k: torch.stack([x[i] for x in images]) for i, k in enumerate(("rgb", "depth", "alpha"))}
    if train:
        torch.autograd.backward([f[k] for f in full for k in ("means", "cov", "opacity", "sh")],
                                [torch.zeros_like(c[k]) if c[k].grad is None else c[k].grad for c in cut
                                 for k in ("means", "cov", "opacity", "sh")])
        out["grads"] = [p.grad for p in leaves[0]]
        if av is not None:
            out["avatar"] = [p.grad for p in leaves[1]]
    return out


def _exact_skin(case, seed):
    s = prepare(case, seed)
    names = ("means", "log_scales", "quats", "joint_idx", "weights", "avatar_of")
    av = _to64(dict(zip(names, s["args"])))
    skin = s["args"][6].to(F).requires_grad_(True)
    leaves = [av[k].requires_grad_(True) for k in names[:3]]
    means, cov = _pose64(av, skin)
    cov6 = torch.stack([cov[:, i, j] for i, j in SIX], 1)
    ((means * s["d_out"][0].to(F)).sum() + (cov6 * s["d_out"][1].to(F)).sum()).backward()
    return {"means": means.detach(), "cov6": cov6.detach(), "d_means": leaves[0].grad, "d_log_scales": leaves[1].grad,
            "d_quats": leaves[2].grad, "d_skin": skin.grad}


def _exact_clearance(case, seed):
    """Distance of each agent's upright axis to every capsule axis, less the radii."""
    s = _to64(prepare(case, seed))
    f = s["at"].floor().clamp(0, 28)
    t, i = (s["at"] - f)[:, None, None], s["first"].long() + f.long()
    caps = ((1 - t) * s["caps"][i] + t * s["caps"][i + 1]).reshape(-1, 8)
    p, q = s["pos"][:, None], caps[None]
    d1 = torch.tensor([0.0, 0.0, HEIGHT], dtype=F, device=DEV)
    d2, r = q[..., 4:7] - q[..., :3], p - q[..., :3]
    a, e, b, c, g = (d1 * d1).sum(), (d2 * d2).sum(-1), (d1 * d2).sum(-1), (d1 * r).sum(-1), (d2 * r).sum(-1)
    best = None
    # the closest points: inside both axes, or at an end of one of them
    x = ((b * g - c * e) / (a * e - b * b).clamp(min=1e-18)).clamp(0, 1)
    for x in (x, torch.zeros_like(x), torch.ones_like(x)):
        y = ((b * x + g) / e).clamp(0, 1)
        x = ((b * y - c) / a).clamp(0, 1)
        dist = (r + x[..., None] * d1 - y[..., None] * d2).norm(dim=-1)
        best = dist if best is None else torch.minimum(best, dist)
    for y in (0.0, 1.0):
        x = ((b * y - c) / a).clamp(0, 1)
        best = torch.minimum(best, (r + x[..., None] * d1 - y * d2).norm(dim=-1))
    return (best - RADIUS - q[..., 3]).min(1).values


def exact(case, seed):
    kind = case["kind"]
    if kind == "sensor":
        s = prepare(case, seed)
        a, d = s["alpha"].to(F), s["depth"].to(F)
        z = torch.where(a > 0, d / a.clamp(min=1e-12), torch.zeros_like(d))
        if case["mesh"]:  # the nearer fragment, by its 32-bit depth
            m = s["mesh_depth"]
            z = torch.where((m > 0) & ~((a > 0) & (z.float() < m)), m.to(F), z)
        return {"rgba": None, "depth": z}
    if kind == "capsules":
        return {"clearance": _exact_clearance(case, seed), "nearest": None, "gap": None, "blocked": None}
    if kind == "skin":
        return _exact_skin(case, seed)
    return _exact_images(case, seed)
