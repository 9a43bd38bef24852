"""Performance cases of the convex hull framework.

Every case is one call (or one forward and backward) through the public
Python entry points of ``paper_1205_1171_amd``, on seeded synthetic inputs
made on the GPU.  Kinds:

  hull       one int32 cloud, faces and status in the caller's buffers (async)
  hull_f32   one float32 cloud snapped to the 30-bit lattice (checked faces)
  batch      many clouds in one call (eager, caller's face buffer)
  replay     many clouds of a fixed layout, one captured call replayed
  delaunay   planar points lifted onto the wide coordinate range
  volume     volume and area of closed surfaces, forward and backward
  adjacency  half-edge twins of a closed surface

Face counts depend on the points, so faces come back in buffers of the
largest size (two rows per point; zero past the faces), with their count.
"""
import math
import random

import numpy as np
import torch

from paper_1205_1171_amd import autograd, autotune, hull

R20 = 1 << 20


def listed():
    return [
        # the smallest call: a collision or packing query on one small body,
        # launches and latency only
        {"name": "hull_97", "kind": "hull", "shape": "cube", "n": 97, "lower": False},
        # the small benchmark cloud: uniform in a cube, few hull vertices
        {"name": "hull_cube_4096", "kind": "hull", "shape": "cube", "n": 4096, "lower": False},
        # a scan of a convex surface, terrain-like use of the lower hull alone,
        # odd size
        {"name": "lower_sphere_60001", "kind": "hull", "shape": "sphere", "n": 60001,
         "lower": True},
        # every point on the hull: the largest output for its input
        {"name": "hull_sphere_1m", "kind": "hull", "shape": "sphere", "n": 1 << 20,
         "lower": False},
        # the benchmark's headline: 99% Gaussian, 1% on an enclosing sphere
        {"name": "hull_mix_16m", "kind": "hull", "shape": "mix", "n": 1 << 24, "lower": False},
        # float32 input (a uniform ball: almost every point is interior), odd size
        {"name": "hull_f32_ball_1m", "kind": "hull_f32", "shape": "ball", "n": (1 << 20) - 3,
         "bits": 30},
        # many small bodies in one eager call (collision shapes, fragments)
        {"name": "batch_20000_small", "kind": "batch", "shape": "both", "clouds": 20000, "lo": 16,
         "hi": 128},
        # the ragged batch workload: sizes from 8 to 65,535, balls and spheres,
        # replayed from one captured graph
        {"name": "replay_10000_ragged", "kind": "replay", "shape": "both", "clouds": 10000, "lo": 8,
         "hi": 65536},
        # equal clouds with radial noise (the differentiable workload's hulls)
        {"name": "batch_256x16384", "kind": "batch", "shape": "noisy", "clouds": 256, "lo": 16384,
         "hi": 16384},
        # Delaunay triangulation of scattered planar samples, odd size
        {"name": "delaunay_262139", "kind": "delaunay", "n": 262139, "half": 1 << 14},
        # volume and area with gradients: one optimisation step's worth
        {"name": "volume_256", "kind": "volume", "clouds": 256, "rings": 96, "segs": 83,
         "inner": 8000},
        # connectivity of a large hull
        {"name": "adjacency_2m", "kind": "adjacency", "rings": 1021, "segs": 1027},
    ]


def _log_int(rng, lo, hi):
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))
    return min(max(v, lo), hi)


def draw(rng: random.Random):
    kind = rng.choice(["hull", "hull", "hull", "hull_f32", "batch", "batch", "replay", "delaunay",
                       "volume", "adjacency"])
    if kind == "hull":
        shape = rng.choice(["cube", "sphere", "ball", "mix"])
        n = _log_int(rng, 64, 1 << 24 if shape == "mix" else 1 << 20)
        return {"kind": kind, "shape": shape, "n": n, "lower": rng.random() < 0.25}
    if kind == "hull_f32":
        return {"kind": kind, "shape": rng.choice(["cube", "sphere", "ball"]),
                "n": _log_int(rng, 64, 1 << 20), "bits": rng.choice([20, 24, 30])}
    if kind in ("batch", "replay"):
        lo = _log_int(rng, 8, 16384)
        hi = _log_int(rng, lo, min(65536, 32 * lo))
        clouds = _log_int(rng, 16, max(16, min(20000, (1 << 23) // hi)))
        return {"kind": kind, "shape": rng.choice(["cube", "sphere", "ball", "both", "noisy"]),
                "clouds": clouds, "lo": lo, "hi": hi}
    if kind == "delaunay":
        return {"kind": kind, "n": _log_int(rng, 64, 1 << 18), "half": 1 << rng.choice([14, 17, 20])}
    if kind == "volume":
        rings, segs = _log_int(rng, 4, 120), _log_int(rng, 5, 120)
        return {"kind": kind, "clouds": _log_int(rng, 1, 256), "rings": rings, "segs": segs,
                "inner": rng.randrange(0, rings * segs + 1)}
    return {"kind": kind, "rings": _log_int(rng, 8, 1021), "segs": _log_int(rng, 8, 1027)}


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _unit(g, n):
    d = torch.randn((n, 3), device="cuda", generator=g, dtype=torch.float64)
    return d / d.norm(dim=1, keepdim=True).clamp_min(1e-300)


def _cloud(shape, n, g, radius=float(R20)):
    """float64 rows of one shape, |c| <= radius (noisy: 5 sigma above it at
    most, in earnest)."""
    if shape == "cube":
        return (torch.rand((n, 3), device="cuda", generator=g, dtype=torch.float64) * 2 - 1) * radius
    if shape == "sphere":
        return _unit(g, n) * radius
    if shape == "ball":
        r = torch.rand((n, 1), device="cuda", generator=g, dtype=torch.float64) ** (1.0 / 3.0)
        return _unit(g, n) * r * radius
    if shape == "noisy":
        r = 1 + torch.randn((n, 1), device="cuda", generator=g, dtype=torch.float64) / 256
        return _unit(g, n) * r * (radius / 4)
    if shape == "mix":
        p = torch.randn((n, 3), device="cuda", generator=g, dtype=torch.float64) * (radius / 16)
        p.clamp_(-radius, radius)
        k = max(n // 100, 1)
        at = torch.randperm(n, device="cuda", generator=g)[:k]
        p[at] = _unit(g, k) * radius
        return p
    raise ValueError(shape)


def _lattice(p):
    return p.round().to(torch.int32).contiguous()


def _batch(case, seed):
    """Points and offsets of a ragged batch (the layout is the case's, the
    points are the seed's); shape "both": ball or sphere, one or the other per
    cloud."""
    lo, hi, H = case["lo"], case["hi"], case["clouds"]
    rs = np.random.RandomState(H * 31 + lo * 7 + hi)
    sizes = np.exp(rs.uniform(math.log(lo), math.log(hi), size=H)).astype(np.int64).clip(lo, hi)
    off = np.zeros(H + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    g = _gen(seed)
    n = int(off[-1])
    if case["shape"] == "both":
        ball = torch.from_numpy(np.repeat(rs.randint(0, 2, size=H), sizes)).to("cuda")
        r = torch.rand((n,), device="cuda", generator=g, dtype=torch.float64) ** (1.0 / 3.0)
        r = torch.where(ball != 0, r, torch.ones_like(r))
        p = _unit(g, n) * (r[:, None] * R20)
    else:
        p = _cloud(case["shape"], n, g)
    return _lattice(p), off


def _surface(rings, segs, g, inner):
    """A closed convex-like surface of rings * segs + 2 vertices with radial
    noise, plus `inner` points inside; rows in random order, faces outward and
    in the order the hull gives them (lower then upper, by slope)."""
    V = rings * segs + 2
    th = (torch.arange(rings, device="cuda", dtype=torch.float64) + 1) * (math.pi / (rings + 1))
    ph = torch.arange(segs, device="cuda", dtype=torch.float64) * (2 * math.pi / segs)
    st = torch.sin(th)[:, None]
    ring = torch.stack([st * torch.cos(ph), st * torch.sin(ph),
                        torch.cos(th)[:, None].expand(rings, segs)], dim=2).reshape(-1, 3)
    poles = torch.tensor([[0.0, 0.0, 1.0], [0.0, 0.0, -1.0]], device="cuda", dtype=torch.float64)
    p = torch.cat([ring, poles])
    p = p * (1 + torch.randn((V, 1), device="cuda", generator=g, dtype=torch.float64) / 4096)
    p = torch.cat([p, _unit(g, inner) * 0.7]) * (1 << 18)
    i = torch.arange(rings - 1, device="cuda")[:, None] * segs
    j = torch.arange(segs, device="cuda")[None, :]
    j1 = (j + 1) % segs
    a, b, c, d = (i + j, i + j1, i + segs + j, i + segs + j1)
    top, bot = V - 2, V - 1
    last = (rings - 1) * segs
    jj, jj1 = j.reshape(-1), j1.reshape(-1)
    f = torch.cat([
        torch.stack([a, c, d], dim=2).reshape(-1, 3), torch.stack([a, d, b], dim=2).reshape(-1, 3),
        torch.stack([torch.full_like(jj, top), jj, jj1], dim=1),
        torch.stack([torch.full_like(jj, bot), last + jj1, last + jj], dim=1)])
    nrm = torch.cross(p[f[:, 1]] - p[f[:, 0]], p[f[:, 2]] - p[f[:, 0]], dim=1)
    up = nrm[:, 2] > 0
    slope = nrm[:, 1] / nrm[:, 2].abs().clamp_min(1e-300)
    key = torch.atan(slope) + up.double() * 10.0
    f = f[torch.argsort(key)]
    perm = torch.randperm(V + inner, device="cuda", generator=g)
    q = torch.empty_like(p)
    q[perm] = p
    return q.float(), perm[f].to(torch.int32)


def _face_buffer(n):
    return torch.zeros((2 * n, 3), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind == "hull":
        n = case["n"]
        x = _lattice(_cloud(case["shape"], n, g))
        ws = hull.Workspace()
        ws.get(hull.workspace_bytes(n), x.device)
        return {"case": case, "x": x, "ws": ws, "faces": _face_buffer(n),
                "info": torch.zeros(2, dtype=torch.int64, device="cuda")}
    if kind == "hull_f32":
        x = _cloud(case["shape"], case["n"], g, 1.0).float().contiguous()
        ws = hull.Workspace()
        ws.get(hull.workspace_bytes(case["n"], hull.WS_F32), x.device)
        return {"case": case, "x": x, "ws": ws, "faces": _face_buffer(case["n"])}
    if kind in ("batch", "replay"):
        x, off = _batch(case, seed)
        schedule = autotune.lookup(off)
        if kind == "replay":
            bh = hull.BatchedHull(x, off, schedule=schedule)
            bh.faces.zero_()
            bh.capture()
            return {"case": case, "bh": bh}
        ws = hull.Workspace()
        ws.get(hull.workspace_bytes_batched(int(off[-1]), case["clouds"]), x.device)
        return {"case": case, "x": x, "off": torch.from_numpy(off), "ws": ws, "schedule": schedule,
                "faces": _face_buffer(len(x))}
    if kind == "delaunay":
        h = case["half"]
        x = torch.randint(-h, h + 1, (case["n"], 2), device="cuda", generator=g, dtype=torch.int32)
        return {"case": case, "x": x, "ws": hull.Workspace(), "faces": _face_buffer(case["n"])}
    if kind == "volume":
        parts = [_surface(case["rings"], case["segs"], g, case["inner"])
                 for _ in range(case["clouds"])]
        po = np.cumsum([0] + [len(q) for q, _ in parts]).astype(np.int64)
        fo = np.cumsum([0] + [len(f) for _, f in parts]).astype(np.int64)
        H = case["clouds"]
        return {"case": case, "p": torch.cat([q for q, _ in parts]).requires_grad_(True),
                "pt_off": torch.from_numpy(po).cuda(),
                "faces": torch.cat([f for _, f in parts]), "face_off": torch.from_numpy(fo).cuda(),
                "gV": torch.rand(H, device="cuda", generator=g) / (1 << 18),
                "gA": torch.rand(H, device="cuda", generator=g)}
    if kind == "adjacency":
        _, f = _surface(case["rings"], case["segs"], g, 0)
        return {"case": case, "faces": f.contiguous(), "ws": hull.Workspace()}
    raise ValueError(kind)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "hull":
        return hull.hull(state["x"], lower_only=case["lower"], ws=state["ws"], faces=state["faces"],
                         info=state["info"])
    if kind in ("hull_f32", "delaunay"):
        if kind == "hull_f32":
            f = hull.hull_f32(state["x"], bits=case["bits"], ws=state["ws"])
        else:
            f = hull.delaunay(state["x"], ws=state["ws"])
        state["faces"][:len(f)] = f  # kept by the caller
        return state["faces"], len(f)
    if kind == "batch":
        return hull.hull_batched(state["x"], state["off"], schedule=state["schedule"],
                                 ws=state["ws"], faces=state["faces"])
    if kind == "replay":
        bh = state["bh"]
        bh.replay()
        return bh.faces, bh.face_off, bh.info
    if kind == "volume":
        V, A = autograd.volume_area(state["p"], state["pt_off"], state["faces"], state["face_off"])
        (gp,) = torch.autograd.grad((V, A), state["p"], (state["gV"], state["gA"]))
        return V, A, gp
    return hull.face_adjacency(state["faces"], ws=state["ws"])


# ---------------------------------------------------------------------------
# Work: the input read once, the faces written once, one orientation (about 14
# operations) per point and per face.
# ---------------------------------------------------------------------------
def _faces(shape, n):
    """About the number of hull faces of n points of a shape."""
    v = {"sphere": n, "noisy": 0.3 * n, "mix": 0.01 * n + 8, "ball": 4.0 * math.sqrt(n),
         "cube": 3.0 * math.log(n + 2) ** 2, "both": 0.5 * n + 2 * math.sqrt(n)}[shape]
    return max(2, 2 * min(v, n) - 4)


def work(case):
    kind = case["kind"]
    if kind in ("hull", "hull", "hull_f32"):
        n, F = case["n"], _faces(case["shape"], case["n"])
        if case.get("lower"):
            F /= 2
        return {"bytes": 12 * n + 12 * F, "flops": 14 * (n + F)}
    if kind in ("batch", "replay"):
        lo, hi, H = case["lo"], case["hi"], case["clouds"]
        m = lo if hi <= lo else (hi - lo) / math.log(hi / lo)  # mean size
        F = _faces(case["shape"], m)
        return {"bytes": H * (12 * m + 12 * F + 16), "flops": 14 * H * (m + F)}
    if kind == "delaunay":
        n = case["n"]
        return {"bytes": 8 * n + 24 * n, "flops": 14 * 3 * n}
    V = case["rings"] * case["segs"] + 2
    F = 2 * V - 4
    if kind == "volume":
        H, N = case["clouds"], V + case["inner"]
        # positions and faces in, gradients out; about 40 operations per face
        # forward and 80 backward
        return {"bytes": H * (24 * N + 12 * F), "flops": H * 120 * F}
    return {"bytes": 24 * F, "flops": 3 * F}


def exact(case, seed):
    """Volume, area and gradient in float64 from the definitions; the other
    kinds return whole numbers."""
    if case["kind"] != "volume":
        return None
    st = prepare(case, seed)
    p = st["p"].detach().double()
    H = case["clouds"]
    counts = (st["face_off"][1:] - st["face_off"][:-1])
    cloud = torch.repeat_interleave(torch.arange(H, device="cuda"), counts)
    f = st["faces"].long() + st["pt_off"][cloud][:, None]
    c = p[st["pt_off"][cloud]]
    a, b, d = p[f[:, 0]], p[f[:, 1]], p[f[:, 2]]
    n = torch.cross(b - a, d - a, dim=1)
    area = n.norm(dim=1)
    vol = ((a - c) * torch.cross(b - c, d - c, dim=1)).sum(dim=1)
    V = torch.zeros(H, dtype=torch.float64, device="cuda").index_add_(0, cloud, vol) / 6
    A = torch.zeros(H, dtype=torch.float64, device="cuda").index_add_(0, cloud, area) / 2
    unit = n / area.clamp_min(1e-300)[:, None]
    gV, gA = st["gV"].double()[cloud][:, None], st["gA"].double()[cloud][:, None]
    grad = torch.zeros_like(p)
    for k, e in ((0, b - d), (1, d - a), (2, a - b)):
        grad.index_add_(0, f[:, k], gV * n / 6 + gA * torch.cross(e, unit, dim=1) / 2)
    return V, A, grad
