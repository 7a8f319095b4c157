"""Timed workloads of the library, through its public entry points.

Each case is a dict of plain values; `prepare` makes its inputs on the GPU from
the case and a seed (a luminaire tree, rays, shading points, a surrogate),
`run` is one call as a program makes it, `exact` the same result in 64 bits
with plain torch.  Luminaires are blob fields like those of the inputs
package (16 Gaussian blobs in log-density and thin shells, float32), drawn on
the GPU so that a large tree is ready in a second.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2207_05009_amd import lumiq

L_MAX = 2048.0
SIGMA_MIN, ALPHA_MAX = 0.1, 0.9
LOG_BASE = math.log(1e-3)
LOG_PRUNE = math.log(0.01)
SIGMA_CLAMP = 50.0
BACKGROUND = (0.05, 0.05, 0.08)
DEV = "cuda"


# --------------------------------------------------------------------- cases
def listed():
    return [
        # interactive picking, a few probes per frame: latency and launches
        dict(name="query_4k_f32", kind="query", rays="sphere", n=4096, depth=6, deg=2, storage="f32",
             model="linear"),
        # the headline: one rendered frame of the depth-9 luminaire
        dict(name="camera_2048_f32", kind="camera", w=2048, h=2048, depth=9, deg=2, storage="f32", model="linear"),
        # a small preview: odd width and height, half storage, SH degree 3, Beer-Lambert
        dict(name="camera_1283x721_f16_exp", kind="camera", w=1283, h=721, depth=8, deg=3, storage="f16",
             model="exp"),
        # next-event estimation from all over a room: incoherent rays, an odd count
        dict(name="room_4m_f16", kind="query", rays="room", n=4194301, depth=9, deg=2, storage="f16",
             model="linear"),
        # a scene with several luminaires, uneven ray counts, one launch
        dict(name="multi_12_f16", kind="multi", trees=12, n=3000017, depth_lo=6, depth_hi=8, deg=3, storage="f16",
             model="linear"),
        # direct light on a floor: uniform samples of the proxy
        dict(name="floor_512_s16", kind="floor", nx=512, ny=512, samples=16, depth=9, deg=2, storage="f32",
             model="linear"),
        # the same with the directional guide
        dict(name="guided_512_s16", kind="guided", nx=512, ny=512, samples=16, grid=16, dirs=2, defensive=0.5,
             depth=8, deg=2, storage="f32", model="linear"),
        # surrogate with octree fallback on room rays
        dict(name="hybrid_4m", kind="hybrid", n=4194301, depth=8, deg=2, storage="f32"),
        # surrogate alone
        dict(name="forward_4m", kind="forward", n=4194301),
        # a slice of surrogate training between two looks at the loss
        dict(name="train_64k_x16", kind="train", batch=65536, steps=16),
        # distillation of a field at 256^3, 256 samples per kept voxel
        dict(name="distill_d8", kind="distill", depth=8, samples=256, blobs=16, shells=4, deg=2),
        # the octree over distilled leaves: built, then its tables saved
        dict(name="build_d8_f16", kind="build", depth=8, deg=2, storage="f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "camera", "camera", "multi", "floor", "guided", "hybrid", "forward", "train",
                       "distill", "build"])
    storage, model = rng.choice(["f32", "f16", "bf16"]), rng.choice(["linear", "linear", "exp"])
    if kind == "query":
        return dict(kind=kind, rays=rng.choice(["sphere", "room"]), n=_log_int(rng, 1, 4 << 20),
                    depth=rng.randint(5, 9), deg=rng.randint(0, 4), storage=storage, model=model)
    if kind == "camera":
        return dict(kind=kind, w=_log_int(rng, 16, 2048), h=_log_int(rng, 16, 2048), depth=rng.randint(6, 9),
                    deg=rng.randint(0, 4), storage=storage, model=model)
    if kind == "multi":
        return dict(kind=kind, trees=rng.randint(2, 16), n=_log_int(rng, 1000, 3 << 20), depth_lo=5, depth_hi=8,
                    deg=rng.randint(2, 3), storage=storage, model=model)
    if kind in ("floor", "guided"):
        nx, ny = _log_int(rng, 8, 512), _log_int(rng, 8, 512)
        c = dict(kind=kind, nx=nx, ny=ny, samples=_log_int(rng, 1, 64), depth=rng.randint(6, 8), deg=2,
                 storage=storage, model=model)
        if c["nx"] * c["ny"] * c["samples"] > 4 << 20:
            c["samples"] = max(1, (4 << 20) // (nx * ny))
        if kind == "guided":
            c.update(grid=_log_int(rng, 1, 32), dirs=rng.randint(1, 4), defensive=round(rng.uniform(0.1, 1.0), 2))
        return c
    if kind == "hybrid":
        return dict(kind=kind, n=_log_int(rng, 100, 4 << 20), depth=rng.randint(6, 8), deg=2, storage=storage)
    if kind == "forward":
        return dict(kind=kind, n=_log_int(rng, 1, 4 << 20))
    if kind == "train":
        return dict(kind=kind, batch=64 * _log_int(rng, 1, 1024), steps=rng.randint(1, 16))
    if kind == "distill":
        return dict(kind=kind, depth=rng.randint(5, 8), samples=_log_int(rng, 8, 256), blobs=rng.randint(1, 32),
                    shells=rng.randint(0, 8), deg=rng.randint(0, 4))
    return dict(kind=kind, depth=rng.randint(5, 8), deg=rng.randint(0, 4), storage=storage)


# -------------------------------------------------------------------- fields
def _field(seed, depth, blobs=16, shells=4, deg=2, occupancy=0.04, shape=None):
    """Parameters of a luminaire's continuous field, as inputs.trees draws
    them; the blobs' common scale is solved for the target occupancy.  With
    `shape` the geometry is that of seed `shape`, and only the light is
    seeded (results then keep their sizes from seed to seed)."""
    rng, light = np.random.default_rng(seed if shape is None else shape), np.random.default_rng(seed + 1000003)
    K = (deg + 1) ** 2
    p = dict(centres=rng.uniform(-0.7, 0.7, (blobs, 3)), amps=rng.uniform(0.5, 1.0, blobs) * math.log(5e4),
             emission=10.0 ** light.uniform(-2.0, 3.0, (blobs, 1)) * light.uniform(0.2, 1.0, (blobs, 3)),
             hi=light.normal(0.0, 0.5, (blobs, 3, K - 1)), shell_half_width=2.0 / (1 << depth), log_base=LOG_BASE,
             sigma_max=SIGMA_CLAMP, l_max=L_MAX, sh_degree=deg)
    u = rng.uniform(0.08, 0.3, blobs)
    p["shells"] = np.concatenate([rng.uniform(-0.5, 0.5, (shells, 3)), rng.uniform(0.25, 0.6, (shells, 1))], 1)
    lo, hi = 0.05, 8.0
    for _ in range(12):
        p["radii"] = math.sqrt(lo * hi) * u
        frac = float(torch.cat([s >= LOG_PRUNE - LOG_BASE for _, s in _slabs(p, 5, torch.float32)]).float().mean())
        lo, hi = (math.sqrt(lo * hi), hi) if frac < occupancy else (lo, math.sqrt(lo * hi))
    return p


def _dev(x, dtype=torch.float64):
    return torch.as_tensor(np.asarray(x), dtype=dtype, device=DEV)


def _slabs(p, depth, dtype):
    """sum_k a_k g_k at every cell centre, slab by slab of z: (z0, [dz, y, x])."""
    n = 1 << depth
    xs = -1.0 + (torch.arange(n, dtype=dtype, device=DEV) + 0.5) * (2.0 / n)
    c, r = _dev(p["centres"], dtype), _dev(p["radii"], dtype)
    g = torch.exp(-(xs[None, None, :] - c[:, :, None]) ** 2 / (2.0 * r * r)[:, None, None])     # [blob, axis, n]
    plane = (g[:, 1, :, None] * g[:, 0, None, :]).reshape(len(r), -1)
    az = (_dev(p["amps"], dtype)[:, None] * g[:, 2]).t().contiguous()
    dz = max(1, min(n, (1 << 24) // (n * n)))
    for z0 in range(0, n, dz):
        yield z0, (az[z0: z0 + dz] @ plane).reshape(-1, n, n)


def _spread(v):
    v = v.to(torch.int64)
    for s, m in ((16, 0x030000FF), (8, 0x0300F00F), (4, 0x030C30C3), (2, 0x09249249)):
        v = (v | (v << s)) & m
    return v


def _compact(v):
    v = v & 0x09249249
    for s, m in ((2, 0x030C30C3), (4, 0x0300F00F), (8, 0x030000FF), (16, 0x000003FF)):
        v = (v | (v >> s)) & m
    return v


def _cells(codes):
    return torch.stack([_compact(codes), _compact(codes >> 1), _compact(codes >> 2)], 1)


def _kept(p, depth, dtype):
    """Morton codes (ascending) of the voxels whose centre density is at least
    the prune threshold, and of those in a shell: codes, log-density, in-shell."""
    n = 1 << depth
    xs = -1.0 + (torch.arange(n, dtype=dtype, device=DEV) + 0.5) * (2.0 / n)
    shells = [[float(v) for v in row] for row in p["shells"]]
    codes, logs, inside = [], [], []
    for z0, s in _slabs(p, depth, dtype):
        sh = torch.zeros_like(s, dtype=torch.bool)
        for cx, cy, cz, rad in shells:
            d = ((xs[z0: z0 + s.shape[0]] - cz) ** 2)[:, None, None] + ((xs - cy) ** 2)[:, None] + (xs - cx) ** 2
            sh |= (d.sqrt() - rad).abs() < p["shell_half_width"]
        z, y, x = torch.nonzero((s >= LOG_PRUNE - LOG_BASE) | sh, as_tuple=True)
        codes.append(_spread(x) | (_spread(y) << 1) | (_spread(z + z0) << 2))
        logs.append(LOG_BASE + s[z, y, x])
        inside.append(sh[z, y, x])
    codes, order = torch.sort(torch.cat(codes))
    return codes, torch.cat(logs)[order], torch.cat(inside)[order]


def _leaves(p, depth):
    """Leaves of a luminaire: codes (int32), density and SH at the centres."""
    codes, logs, inside = _kept(p, depth, torch.float32)
    sigma = torch.where(inside, torch.tensor(SIGMA_CLAMP, device=DEV), torch.exp(logs).clamp_max(SIGMA_CLAMP))
    K = (p["sh_degree"] + 1) ** 2
    sh = torch.empty((len(codes), 3, K), device=DEV)
    c, r = _dev(p["centres"], torch.float32), _dev(p["radii"], torch.float32)
    em, hi = _dev(p["emission"], torch.float32), _dev(p["hi"], torch.float32).reshape(len(r), -1)
    for a in range(0, len(codes), 1 << 21):
        pos = -1.0 + (_cells(codes[a: a + (1 << 21)]).float() + 0.5) * (2.0 / (1 << depth))
        w = torch.softmax(-((pos[:, None] - c) ** 2).sum(-1) / (2.0 * r * r), 1)
        f = (w @ em) / L_MAX
        sh[a: a + len(w), :, 0] = torch.log(f / (1.0 - f)) * (2.0 * math.sqrt(math.pi))
        sh[a: a + len(w), :, 1:] = (w @ hi).reshape(len(w), 3, K - 1)
    return codes.to(torch.int32), sigma.float().contiguous(), sh


def _luminaire(seed, depth, deg, storage, shape=None):
    codes, sigma, sh = _leaves(_field(seed, depth, deg=deg, shape=shape), depth)
    return dict(depth=depth, deg=deg, storage=storage, codes=codes, sigma=sigma, sh=sh)


def _octree(t):
    return lumiq.octree_from_leaves(t["depth"], t["deg"], t["codes"], t["sigma"], t["sh"], L_MAX, SIGMA_MIN, ALPHA_MAX,
                                    t["storage"])


# ---------------------------------------------------------------------- rays
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 13)


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV)


def _unit(v):
    return (v / v.norm(dim=1, keepdim=True)).contiguous()


def _sphere_rays(g, n):
    o = _unit(torch.randn((n, 3), generator=g, device=DEV)) * 3.0
    return o, _unit(2.0 * _rand(g, n, 3) - 1.0 - o)


def _room_rays(g, n):
    """Origins in a 10 x 10 x 3 room outside the proxy, aimed at uniform points of its surface."""
    half = torch.tensor([5.0, 5.0, 1.5], device=DEV)
    o = (2.0 * _rand(g, n, 3) - 1.0) * half
    inside = (o.abs() <= 1.0).all(1)
    o[:, 0] += torch.where(inside, torch.where(o[:, 0] < 0, -1.5, 1.5), 0.0)
    t = 2.0 * _rand(g, n, 3) - 1.0
    face = torch.randint(0, 6, (n,), generator=g, device=DEV)
    t.scatter_(1, (face % 3)[:, None], torch.where(face < 3, 1.0, -1.0)[:, None])
    return o, _unit(t - o)


def _camera_rays(g, w, h):
    """Pinhole at distance 3 from a seeded direction above the horizon, 40 degrees."""
    a, b = (float(v) for v in _rand(g, 2))
    th, ph = math.radians(35.0 + 40.0 * a), 2.0 * math.pi * b
    eye = 3.0 * np.array([math.sin(th) * math.cos(ph), math.sin(th) * math.sin(ph), math.cos(th)])
    fwd = -eye / 3.0
    right = np.cross(fwd, [0.0, 0.0, 1.0])
    right /= np.linalg.norm(right)
    up = np.cross(right, fwd)
    k = math.tan(math.radians(20.0))
    sx = (2.0 * (torch.arange(w, device=DEV) + 0.5) / w - 1.0) * k * w / h
    sy = (1.0 - 2.0 * (torch.arange(h, device=DEV) + 0.5) / h) * k
    f, r, u = (_dev(v, torch.float32) for v in (fwd, right, up))
    d = _unit((f + sx[None, :, None] * r + sy[:, None, None] * u).reshape(-1, 3))
    return _dev(eye, torch.float32).expand(len(d), 3).contiguous(), d


def _floor(nx, ny):
    xs = (torch.arange(nx, device=DEV) + 0.5) / nx * 10.0 - 5.0
    ys = (torch.arange(ny, device=DEV) + 0.5) / ny * 10.0 - 5.0
    p = torch.full((ny, nx, 3), -1.5, device=DEV)
    p[:, :, 0], p[:, :, 1] = xs, ys[:, None]
    p = p.reshape(-1, 3).contiguous()
    return p, torch.tensor([0.0, 0.0, 1.0], device=DEV).expand(len(p), 3).contiguous()


def _pairs(g, n):
    """Training pairs: room rays and a smooth high-dynamic-range radiance."""
    o, d = _room_rays(g, n)
    rgb = torch.exp(2.0 * torch.sin(3.0 * o[:, :1] + 5.0 * d) + o[:, 1:2]).contiguous()
    return o, d, rgb


def _offsets(case, seed):
    r = np.random.default_rng(seed + 5)
    w = np.exp(r.uniform(math.log(1.0), math.log(2000.0), case["trees"]))
    return np.concatenate([[0], np.round(np.cumsum(w) / w.sum() * case["n"])]).astype(np.int64)


# ------------------------------------------------------------------- prepare
def _inputs(case, seed):
    g, k = _gen(seed), case["kind"]
    s = dict(case=case)
    if k in ("query", "camera", "hybrid", "floor", "guided"):
        s["tree"] = _luminaire(seed, case["depth"], case["deg"], case["storage"])
    if k == "query":
        s["o"], s["d"] = (_sphere_rays if case["rays"] == "sphere" else _room_rays)(g, case["n"])
    elif k == "camera":
        s["o"], s["d"] = _camera_rays(g, case["w"], case["h"])
    elif k == "multi":
        depths = np.random.default_rng(seed).integers(case["depth_lo"], case["depth_hi"] + 1, case["trees"])
        s["trees"] = [_luminaire(seed * 100 + i, int(dd), case["deg"], case["storage"]) for i, dd in enumerate(depths)]
        s["offsets"] = _offsets(case, seed)
        s["o"], s["d"] = _room_rays(g, case["n"])
    elif k in ("floor", "guided"):
        s["p"], s["nrm"] = _floor(case["nx"], case["ny"])
        s["u"] = _rand(g, len(s["p"]), case["samples"], 3)
        if k == "guided":
            m = 6 * case["grid"] ** 2 * case["dirs"] ** 2
            s["w"] = -torch.log1p(-_rand(g, m)) * (_rand(g, m) > 0.3)
    elif k in ("hybrid", "forward"):
        s["o"], s["d"] = _room_rays(g, case["n"])
    elif k == "train":
        s["o"], s["d"], s["rgb"] = _pairs(g, case["batch"] * case["steps"] + 37)
    elif k == "distill":
        s["field"] = _field(seed, case["depth"], case["blobs"], case["shells"], case["deg"], shape=10)
        s["seed"] = seed
    elif k == "build":
        s["tree"] = _luminaire(seed, case["depth"], case["deg"], case["storage"], shape=10)
    if k in ("hybrid", "forward", "train"):
        s["theta"] = _theta(seed)
    return s


def _theta(seed):
    """He-uniform weights and small biases (so that a bias gradient matters), float32."""
    r = np.random.default_rng(seed + 31)
    parts = []
    for i, o in ((128, 64), (64, 64), (64, 64), (64, 64), (64, 3)):
        parts += [r.uniform(-1.0, 1.0, i * o) * math.sqrt(6.0 / i), r.uniform(-0.1, 0.1, o)]
    return np.concatenate(parts).astype(np.float32)


def prepare(case, seed):
    s, k = _inputs(case, seed), case["kind"]
    if k in ("query", "camera", "hybrid", "floor", "guided"):
        s["oct"] = _octree(s["tree"])
    if k == "multi":
        s["octs"] = [_octree(t) for t in s["trees"]]
    if k in ("query", "camera", "multi", "hybrid", "forward"):
        s["rgb_out"] = torch.empty_like(s["o"])
        s["alpha_out"] = torch.empty(len(s["o"]), device=DEV)
    if k in ("floor", "guided"):
        s["E"] = torch.empty_like(s["p"])
    if k in ("hybrid", "forward", "train"):
        s["net"] = lumiq.Surrogate(seed=31)
        s["net"].set_params(s["theta"])
    if k == "hybrid":
        # held-out pairs: the network is right about lines that head down
        # where they enter low, and wrong about the others it is asked for,
        # so that about half of the room's bins are trusted
        o, d = _room_rays(_gen(seed + 1), 1 << 25)
        ref = s["net"].forward(o, d)
        ref[(d[:, 0] * o[:, 1] > 1.0)] *= 3.0
        s["net"].build_trust(o, d, ref)
    s.pop("tree" if k != "build" else "", None)
    s.pop("trees", None)
    return s


# ----------------------------------------------------------------------- run
def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "query":
        return s["oct"].query(s["o"], s["d"], model=c["model"], rgb=s["rgb_out"], alpha=s["alpha_out"])
    if k == "camera":
        return s["oct"].query_image(s["o"], s["d"], c["w"], c["h"], model=c["model"], rgb=s["rgb_out"],
                                    alpha=s["alpha_out"])
    if k == "multi":
        return lumiq.query_multi(s["octs"], s["offsets"], s["o"], s["d"], model=c["model"], rgb=s["rgb_out"],
                                 alpha=s["alpha_out"])
    if k == "floor":
        return s["oct"].proxy_irradiance(s["p"], s["nrm"], s["u"], background=BACKGROUND, model=c["model"],
                                         irradiance=s["E"])[0]
    if k == "guided":
        return s["oct"].proxy_irradiance_guided(s["p"], s["nrm"], s["u"], s["w"], c["grid"], c["defensive"],
                                                background=BACKGROUND, model=c["model"], irradiance=s["E"],
                                                dir_res=c["dirs"])[0]
    if k == "hybrid":
        return s["net"].infer(s["o"], s["d"], s["oct"], rgb=s["rgb_out"])
    if k == "forward":
        return s["net"].forward(s["o"], s["d"], rgb=s["rgb_out"])
    if k == "train":
        losses = s["net"].train(s["o"], s["d"], s["rgb"], steps=c["steps"], total_steps=20000, batch=c["batch"])
        return losses, s["net"].get_params()
    if k == "distill":
        codes, sigma, sh = lumiq.distill_leaves(s["field"], c["depth"], 0.01, c["samples"], seed=s["seed"])
        return dict(codes=codes, sigma=sigma, sh=sh)
    tree = _octree(s["tree"])
    tables = tree.download()
    tree.free()
    return tables


# ---------------------------------------------------------------------- work
MLP_FLOP = 2 * (128 * 64 + 3 * 64 * 64 + 64 * 3)


def work(case):
    """Bytes that have to move (each input read once, each output written once) and operations.

    A query has to read its rays and write radiance and opacity; how much of
    the tree it touches depends on the view and is not counted.
    """
    k = case["kind"]
    if k in ("query", "multi"):
        return dict(bytes=40 * case["n"], flops=0)
    if k == "camera":
        return dict(bytes=40 * case["w"] * case["h"], flops=0)
    if k in ("floor", "guided"):
        return dict(bytes=case["nx"] * case["ny"] * (36 + 12 * case["samples"]), flops=0)
    if k == "hybrid":
        return dict(bytes=37 * case["n"], flops=0)
    if k == "forward":
        return dict(bytes=36 * case["n"], flops=MLP_FLOP * case["n"])
    if k == "train":
        n = case["batch"] * case["steps"]
        return dict(bytes=36 * n + 24 * 20931 * case["steps"], flops=3 * MLP_FLOP * n)
    K = (case["deg"] + 1) ** 2
    if k == "distill":
        # about 5% of the voxels are kept; per sample and blob 23 operations
        kept = 0.05 * 8 ** case["depth"]
        return dict(bytes=kept * (8 + 12 * K), flops=kept * case["samples"] * (24 + 23 * case["blobs"]))
    kept = 0.05 * 8 ** case["depth"]
    return dict(bytes=kept * (8 + 12 * K) * 2, flops=0)


# --------------------------------------------------------------- in 64 bits
def _sh64(deg, w):
    """Real orthonormal SH without the Condon-Shortley phase, [n, (deg + 1)^2]."""
    x, y, z = w.unbind(1)
    out = [None] * (deg + 1) ** 2
    c, s = torch.ones_like(x), torch.zeros_like(x)          # rho^m cos(m phi), rho^m sin(m phi)
    for m in range(deg + 1):
        p0, p1 = None, torch.full_like(x, float(math.prod(range(1, 2 * m, 2))))
        for l in range(m, deg + 1):
            if l > m:
                p0, p1 = p1, ((2 * l - 1) * z * p1 - (0.0 if p0 is None else (l + m - 1) * p0)) / (l - m)
            k = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - m) / math.factorial(l + m))
            if m == 0:
                out[l * l + l] = k * p1
            else:
                out[l * l + l + m], out[l * l + l - m] = (math.sqrt(2) * k * p1 * v for v in (c, s))
        c, s = x * c - y * s, x * s + y * c
    return torch.stack(out, 1)


class _Grid64:
    """The stored tree as dense grids: leaf index per finest cell, occupancy per level."""

    def __init__(self, t):
        ty = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[t["storage"]]
        self.sigma, self.sh = t["sigma"].to(ty).double(), t["sh"].to(ty)
        self.D, self.deg, n = t["depth"], t["deg"], 1 << t["depth"]
        keep = torch.nonzero(t["sigma"].to(ty).float() >= torch.tensor(SIGMA_MIN, device=DEV))[:, 0]
        q = _cells(t["codes"].long()[keep])
        self.leaf = torch.full((n, n, n), -1, dtype=torch.int32, device=DEV)
        self.leaf[q[:, 2], q[:, 1], q[:, 0]] = keep.int()
        self.occ = [None] * (self.D + 1)
        self.occ[self.D] = (self.leaf >= 0)
        for l in range(self.D - 1, -1, -1):
            m = 1 << l
            self.occ[l] = self.occ[l + 1].reshape(m, 2, m, 2, m, 2).any(5).any(3).any(1)


def _query64(t, o32, d32, model, chunk=1 << 21):
    """Radiance and opacity of rays through the stored tree, marched in float64."""
    G = t if isinstance(t, _Grid64) else _Grid64(t)
    n = 1 << G.D
    amax = float(np.float32(ALPHA_MAX))
    rgb, alpha = torch.zeros(len(o32), 3, dtype=torch.float64, device=DEV), torch.zeros(len(o32), dtype=torch.float64,
                                                                                       device=DEV)
    for a in range(0, len(o32), chunk):
        o, d = o32[a: a + chunk].double(), d32[a: a + chunk].double()
        near = (torch.where(d > 0, -1.0, 1.0) - o) / d
        far = (torch.where(d > 0, 1.0, -1.0) - o) / d
        still = d == 0
        near, far = near.masked_fill(still, -math.inf), far.masked_fill(still, math.inf)
        t0 = near.max(1).values.clamp_min(0.0)
        idx = torch.nonzero((t0 < far.min(1).values) & (~still | ((o >= -1) & (o < 1))).all(1))[:, 0]
        o, d, tt = o[idx], d[idx], t0[idx]
        q = ((o + tt[:, None] * d + 1.0) * (n / 2)).floor().clamp(0, n - 1).long()
        Y = _sh64(G.deg, -d / d.norm(dim=1, keepdim=True))
        dl = d.norm(dim=1)
        L, T = torch.zeros_like(o), torch.ones_like(tt)
        while len(idx):
            leaf = G.leaf[q[:, 2], q[:, 1], q[:, 0]].long()
            size = torch.ones_like(leaf)
            empty = leaf < 0
            for l in range(G.D - 1, 0, -1):
                b = q >> (G.D - l)
                empty &= ~G.occ[l][b[:, 2], b[:, 1], b[:, 0]]
                size = torch.where(empty, 1 << (G.D - l), size)
            lo = torch.div(q, size[:, None], rounding_mode="floor") * size[:, None]
            k = torch.where(d > 0, lo + size[:, None], lo)
            tc = ((-1.0 + k.double() * (2.0 / n)) - o) / d
            tc = tc.masked_fill(d == 0, math.inf)
            xt, xa = tc.min(1)
            at = torch.nonzero(leaf >= 0)[:, 0]
            lf = leaf[at]
            sd = G.sigma[lf] * ((xt - tt)[at].clamp_min(0.0) * dl[at])
            w = torch.minimum(sd, T[at]) if model == "linear" else -T[at] * torch.expm1(-sd)
            x = (G.sh[lf].double() * Y[at][:, None]).sum(-1)
            L[at] += w[:, None] * (L_MAX * torch.sigmoid(x))
            T[at] -= w
            g = ((o + xt[:, None] * d + 1.0) * (n / 2)).floor().long()
            g = torch.minimum(torch.maximum(g, lo), lo + size[:, None] - 1)
            step = torch.where(d > 0, lo + size[:, None], lo - 1)
            q = torch.where(torch.arange(3, device=DEV) == xa[:, None], step, g)
            done = ((q < 0) | (q >= n)).any(1) | ((leaf >= 0) & (1.0 - T >= amax))
            rgb[a + idx[done]], alpha[a + idx[done]] = L[done], 1.0 - T[done]
            go = torch.nonzero(~done)[:, 0]
            idx, o, d, tt, q, Y, dl, L, T = (v[go] for v in (idx, o, d, xt, q, Y, dl, L, T))
    return rgb, alpha


def _proxy_points64(f, a, b):
    """Face points (float32 coordinates a, b on face f) and the faces' signed axes."""
    axis, sgn = f // 2, torch.where(f % 2 == 1, 1.0, -1.0)
    y = torch.empty(f.shape + (3,), device=DEV)
    y.scatter_(-1, axis[..., None], sgn[..., None])
    y.scatter_(-1, ((axis + 1) % 3)[..., None], a[..., None])
    y.scatter_(-1, ((axis + 2) % 3)[..., None], b[..., None])
    return y, axis, sgn.double()


def _irradiance64(case, s, f, a, b, inv_density):
    """Mean over the samples of w (L_e + (1 - alpha) L_b), Eq. 2."""
    y, axis, sgn = _proxy_points64(f, a, b)
    x = s["p"][:, None].expand_as(y)
    d = (y - x).contiguous()
    d64, n64 = d.double(), s["nrm"].double()[:, None]
    r2 = (d64 * d64).sum(-1)
    ndot = (n64 * d64).sum(-1) / n64.norm(dim=-1)
    h = sgn * x.double().gather(-1, axis[..., None])[..., 0] - 1.0
    w = torch.where((h > 0) & (ndot > 0), ndot * h / (r2 * r2) * inv_density, 0.0)
    live = torch.nonzero(w.reshape(-1) > 0)[:, 0]
    rgb, alpha = _query64(s["tree"], x.reshape(-1, 3)[live], d.reshape(-1, 3)[live], case["model"])
    terms = torch.zeros(w.numel(), 3, dtype=torch.float64, device=DEV)
    terms[live] = w.reshape(-1)[live, None] * (rgb + (1.0 - alpha)[:, None] * _dev(np.float32(BACKGROUND)))
    return terms.reshape(w.shape + (3,)).mean(1)


def _bins64(v, l2, D):
    """Tangent bin of components v of directions with squared length l2."""
    i = torch.zeros_like(v, dtype=torch.long)
    for j in range(1, D):
        th = 2.0 * j / D - 1.0
        if th < 0:
            ok = (v >= 0) | (v * v <= th * th * l2)
        elif th == 0:
            ok = v >= 0
        else:
            ok = (v >= 0) & (v * v >= th * th * l2)
        i = torch.where(ok, j, i)
    return i


def _guided64(case, s):
    """The guided sampler's choice of cell, as the header states it."""
    grid, D, beta = case["grid"], case["dirs"], float(np.float32(case["defensive"]))
    gg, cells = grid * grid, 6 * grid * grid
    w = s["w"].double().reshape(cells, D * D).t().contiguous()
    W = w.sum(1, keepdim=True)
    p = torch.where(W > 0, (1.0 - beta) * w / W + beta / cells, 1.0 / cells)
    cdf = torch.cat([torch.zeros(D * D, 1, dtype=torch.float64, device=DEV), p.cumsum(1)], 1)
    x, nrm = s["p"].double(), s["nrm"].double()
    P, gf, tab = (torch.zeros(len(x), 6, dtype=v, device=DEV) for v in (torch.float64, torch.float64, torch.long))
    for f in range(6):
        ax, sg = f >> 1, 1.0 if f & 1 else -1.0
        c = torch.zeros(3, dtype=torch.float64, device=DEV)
        c[ax] = sg
        e = c - x
        l2 = (e * e).sum(1)
        tab[:, f] = _bins64(-e[:, (ax + 1) % 3], l2, D) * D + _bins64(-e[:, (ax + 2) % 3], l2, D)
        vis = sg * x[:, ax] > 1.0
        P[:, f] = torch.where(vis, cdf[tab[:, f], (f + 1) * gg] - cdf[tab[:, f], f * gg], 0.0)
        gf[:, f] = torch.where(vis, ((nrm * e).sum(1) * (sg * x[:, ax] - 1.0) / (l2 * l2)).clamp_min(0.0), 0.0)
    S, pv = (P * gf).sum(1, keepdim=True), P.sum(1, keepdim=True)
    Q = torch.where(S > 0, 0.5 * P * gf / S + 0.5 * P / pv, P / pv).nan_to_num(0.0)
    vis = torch.stack([(1.0 if f & 1 else -1.0) * x[:, f >> 1] > 1.0 for f in range(6)], 1)
    last = torch.where(vis, torch.arange(6, device=DEV), -1).max(1).values
    t = s["u"][..., 0].double()
    face = torch.full(t.shape, -1, dtype=torch.long, device=DEV)
    rest = t.clone()
    for f in range(6):
        take = (face < 0) & vis[:, f, None] & ((t < Q[:, f, None]) | (last == f)[:, None])
        face = torch.where(take, f, face)
        rest = torch.where(take, t, rest)
        t = torch.where(face < 0, t - Q[:, f, None] * vis[:, f, None], t)
    fc = face.clamp_min(0)
    Qs, Ps, ts = Q.gather(1, fc), P.gather(1, fc), tab.gather(1, fc)
    target = cdf[ts, fc * gg] + torch.where(Qs > 0, rest / Qs, 0.0) * Ps
    lo, hi = fc * gg, fc * gg + gg - 1
    for _ in range(gg.bit_length() + 1):
        mid = (lo + hi + 1) // 2
        ok = cdf[ts, mid] <= target
        lo, hi = torch.where(ok & (lo < hi), mid, lo), torch.where(ok | (lo >= hi), hi, mid - 1)
    pa = p[ts, lo] * torch.where(Ps > 0, Qs / Ps, 0.0) / (2.0 / grid) ** 2
    inv = torch.where((face >= 0) & (pa > 0), 1.0 / pa, 0.0)
    step = torch.tensor(2.0 / grid, dtype=torch.float32, device=DEV)
    a = (((lo // grid) % grid).float() + s["u"][..., 1]) * step - 1.0
    b = ((lo % grid).float() + s["u"][..., 2]) * step - 1.0
    return _irradiance64(case, s, fc, a, b, inv)


def _layers(theta):
    out, at = [], 0
    for i, o in ((128, 64), (64, 64), (64, 64), (64, 64), (64, 3)):
        out.append((theta[at: at + i * o].reshape(o, i), theta[at + i * o: at + i * o + o]))
        at += i * o + o
    return out


def _features64(o, d):
    """The 126 Fourier features of a ray's line (two zero pads), and whether it meets the sphere."""
    d = d / d.norm(dim=1, keepdim=True)
    b = (o * d).sum(1)
    disc = b * b - ((o * o).sum(1) - 3.0)
    e = (o + (-b - disc.clamp_min(0.0).sqrt())[:, None] * d) / math.sqrt(3.0)
    x = torch.cat([e, d], 1)
    ang = x[:, :, None] * (math.pi * 2.0 ** torch.arange(10, dtype=torch.float64, device=DEV))
    f = torch.cat([x[:, :, None], torch.stack([ang.sin(), ang.cos()], 3).reshape(len(x), 6, 20)], 2).reshape(len(x), 126)
    return torch.nn.functional.pad(f, (0, 2)), disc > 0


def _net64(theta, f):
    ls = _layers(theta)
    for w, b in ls[:-1]:
        f = torch.relu(f @ w.t() + b)
    return f @ ls[-1][0].t() + ls[-1][1]


def _forward64(s):
    theta, out = _dev(s["theta"]), []
    for a in range(0, len(s["o"]), 1 << 19):
        f, hit = _features64(s["o"][a: a + (1 << 19)].double(), s["d"][a: a + (1 << 19)].double())
        out.append(torch.where(hit[:, None], (torch.exp(_net64(theta, f)) - 0.01).clamp_min(0.0), 0.0))
    return torch.cat(out)


def _train64(case, s):
    """The run's first Adam steps in float64: the losses and the weights after them."""
    theta = _dev(s["theta"]).requires_grad_()
    m, v, losses = torch.zeros_like(theta), torch.zeros_like(theta), []
    B, n = case["batch"], len(s["o"])
    for k in range(case["steps"]):
        at = torch.arange(k * B, k * B + B, device=DEV) % n
        f, hit = _features64(s["o"][at].double(), s["d"][at].double())
        L = torch.exp(_net64(theta, f[hit])) - 0.01
        den = L.detach().mean(1, keepdim=True) + 0.01
        loss = (((L - s["rgb"][at][hit].double()) / den) ** 2).sum() / B
        g, = torch.autograd.grad(loss, theta)
        losses.append(float(loss.detach()))
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        lr = 5e-4 * (5e-6 / 5e-4) ** (k / 20000)
        with torch.no_grad():
            theta -= lr * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return np.array(losses), theta.detach()


def _philox64(code, j, key):
    """Philox4x32-10 words of counters (code, j, 0, 0), in int64 arithmetic."""
    m32 = 0xFFFFFFFF

    def mul(a, c):                      # 32 x 32 -> high and low words without 64-bit overflow
        lo, hi = (c & 0xFFFF) * a, (c >> 16) * a
        mid = hi + (lo >> 16)
        return mid >> 16, ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)

    c0, c1 = torch.broadcast_tensors(code, j)
    c2 = c3 = torch.zeros_like(c0)
    k0, k1 = key & m32, key >> 32
    for _ in range(10):
        h0, l0 = mul(c0, 0xD2511F53)
        h1, l1 = mul(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c0, c1, c2


def _distill64(case, s):
    p, h = s["field"], 2.0 / (1 << case["depth"])
    codes, _, _ = _kept(p, case["depth"], torch.float64)
    c, r, a = _dev(p["centres"]), _dev(p["radii"]), _dev(p["amps"])
    em, K = _dev(p["emission"]), (case["deg"] + 1) ** 2
    hi = _dev(p["hi"]).reshape(len(r), -1)
    sigma = torch.zeros(len(codes), dtype=torch.float64, device=DEV)
    sh = torch.zeros(len(codes), 3, K, dtype=torch.float64, device=DEV)
    j = torch.arange(case["samples"], device=DEV)
    step = max(1, (1 << 22) // case["samples"])
    for i in range(0, len(codes), step):
        cc = codes[i: i + step]
        off = torch.stack(_philox64(cc[:, None], j, s["seed"]), -1) >> 8
        x = (-1.0 + _cells(cc).double() * h)[:, None] + off.double() * (2.0 ** -24 * h)
        lw = torch.stack([-((x - c[k]) ** 2).sum(-1) / (2.0 * r[k] * r[k]) for k in range(len(r))], -1)
        sg = torch.exp(p["log_base"] + (a * torch.exp(lw)).sum(-1)).clamp_max(SIGMA_CLAMP)
        for row in p["shells"]:
            dist = (x - _dev(row[:3])).norm(dim=-1)
            sg = torch.where((dist - float(row[3])).abs() < p["shell_half_width"], SIGMA_CLAMP, sg)
        w = torch.softmax(lw, -1)
        f = (w @ em) / L_MAX
        sigma[i: i + step] = sg.mean(1)
        sh[i: i + step, :, 0] = (torch.log(f / (1.0 - f)) * (2.0 * math.sqrt(math.pi))).mean(1)
        sh[i: i + step, :, 1:] = (w.mean(1) @ hi).reshape(-1, 3, K - 1)
    return dict(codes=codes.int(), sigma=sigma, sh=sh)


def _tables64(t):
    ty = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[t["storage"]]
    levels = [t["codes"].long()]
    for _ in range(t["depth"]):
        levels.insert(0, torch.unique_consecutive(levels[0] >> 3))
    base = np.concatenate([[0], np.cumsum([len(v) for v in levels[:-1]])])
    child = torch.zeros(int(base[-1]), 8, dtype=torch.int32, device=DEV)
    for l in range(t["depth"]):
        kids = levels[l + 1]
        i = torch.arange(len(kids), device=DEV)
        child[int(base[l]) + torch.searchsorted(levels[l], kids >> 3), kids & 7] = (
            -1 - i if l + 1 == t["depth"] else int(base[l + 1]) + i).int()
    return dict(child=child, sigma=t["sigma"].to(ty).double(), sh=t["sh"].to(ty).double())


def exact(case, seed):
    k = case["kind"]
    if k == "hybrid":
        return None          # which path answers a ray is decided on float32 bins
    s = _inputs(case, seed)
    if k in ("query", "camera"):
        return _query64(s["tree"], s["o"], s["d"], case["model"])
    if k == "multi":
        off = s["offsets"]
        parts = [_query64(t, s["o"][off[i]: off[i + 1]], s["d"][off[i]: off[i + 1]], case["model"])
                 for i, t in enumerate(s["trees"])]
        return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
    if k == "floor":
        u = s["u"]
        return _irradiance64(case, s, (u[..., 0] * 6.0).long().clamp(0, 5), u[..., 1] * 2.0 - 1.0,
                             u[..., 2] * 2.0 - 1.0, 24.0)
    if k == "guided":
        return _guided64(case, s)
    if k == "forward":
        return _forward64(s)
    if k == "train":
        return _train64(case, s)
    if k == "distill":
        return _distill64(case, s)
    return _tables64(s["tree"])
