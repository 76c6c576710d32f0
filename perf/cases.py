"""The work that a user of this framework has it do, as cases that can be timed.

Scenes are synthetic: a furnace sphere, a box room and a fruit bowl of
Gaussian surfels with the surfel spacing, opacities and albedos of the
workloads this repository is benchmarked on.  A case is a dict of plain
values; ``kind`` says which call (or calls) one pass makes:

step      one optimisation step: BVH, ray-cast form factors, direct light,
          bounces, adjoint, opacity gradient
fixed     bounces and adjoint on an F that stays (relighting, albedo fitting)
serve     the allocation-free bounces of a serving loop
dense     many lights at once, BF16 products on the dense copies of F
batch     rooms of uneven size joined into one operator, forward and backward
hits      opacity and geometry gradients through the recorded hits
sh        directional transfer with the diffuse + Phong BRDF, both directions
center    centre-to-centre form factors and their gradients
mc        Monte-Carlo TD(0) rounds
lights    direct light of many lights and its gradients
"""
import math

import numpy as np
import torch

import paper_2509_18497_amd as g

FIELDS = ("px", "py", "pz", "tux", "tuy", "tuz", "tvx", "tvy", "tvz", "nx", "ny", "nz", "su", "sv", "opacity")
T_MIN = 1e-4


def listed():
    return [
        # the furnace check, the smallest whole step: calls and launches count
        {"name": "step furnace 512", "kind": "step", "scene": "sphere", "n": 512, "R": 64, "topk": 0, "K": 1,
         "bounces": 6, "lights": 1, "autograd": True},
        # a room, every F entry kept, through the autograd function
        {"name": "step room 16k", "kind": "step", "scene": "room", "n": 16384, "R": 256, "topk": 0, "K": 9,
         "bounces": 8, "lights": 1, "autograd": True},
        # the fruit bowl, the full step the framework is benchmarked on
        {"name": "step bowl 100k", "kind": "step", "scene": "bowl", "n": 100000, "R": 128, "topk": 512, "K": 16,
         "bounces": 8, "lights": 1, "autograd": False},
        # the same operator kept while lights or albedo are fitted
        {"name": "fixed bowl 100k", "kind": "fixed", "scene": "bowl", "n": 100000, "R": 128, "topk": 512, "K": 16,
         "bounces": 8, "lights": 1},
        # one relit frame of a small scene in a serving loop
        {"name": "serve sphere 1500", "kind": "serve", "scene": "sphere", "n": 1500, "R": 64, "topk": 64, "K": 4,
         "bounces": 4, "lights": 1},
        # the multi-light room: 100 lights as right-hand sides
        {"name": "dense room 32k", "kind": "dense", "scene": "room", "n": 32768, "R": 256, "topk": 0, "K": 9,
         "bounces": 8, "lights": 100},
        # rooms of uneven size, 8 to 100 lights each
        {"name": "batch 8 rooms", "kind": "batch", "scene": "room", "rooms": 8, "n_lo": 2048, "n_hi": 12288,
         "lights_lo": 8, "lights_hi": 100, "R": 128, "topk": 512, "K": 9, "bounces": 8, "bf16": False},
        # gradients through the recorded hits of a cast
        {"name": "hits bowl 30k", "kind": "hits", "scene": "bowl", "n": 30000, "R": 128, "topk": 512},
        # glossy materials
        {"name": "sh bowl 50k", "kind": "sh", "scene": "bowl", "n": 50000, "R": 128, "topk": 512, "K": 16,
         "bounces": 8, "lights": 1},
        # the centre-to-centre decay with a learnable scale
        {"name": "center bowl 20k", "kind": "center", "scene": "bowl", "n": 20000, "R": 128, "topk": 512},
        # the stochastic solver
        {"name": "mc bowl 50k", "kind": "mc", "scene": "bowl", "n": 50000, "rounds": 16, "K": 4, "lights": 1},
        # light placement: all lights of a capture
        {"name": "lights room 16k", "kind": "lights", "scene": "room", "n": 16384, "K": 9, "lights": 100},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "fixed", "serve", "dense", "batch", "hits", "sh", "center", "mc", "lights"])
    scene = rng.choice(["room", "bowl"])
    c = {"kind": kind, "scene": scene}
    if kind == "step":
        c["n"] = _log(rng, 512, 100000)
        c["R"] = min(rng.choice([64, 100, 128, 256]), max(16, 12800000 // c["n"]))
        c["topk"] = 0 if c["n"] <= 16384 and rng.random() < 0.5 else rng.choice([256, 512])
        c["K"] = rng.choice([1, 4, 9, 16])
        c["bounces"] = rng.randint(3, 8)
        c["lights"] = 1
        c["autograd"] = rng.random() < 0.5
    elif kind == "fixed":
        c["n"] = _log(rng, 2000, 100000)
        c["K"] = rng.choice([1, 4, 9, 16])
        c["lights"] = max(1, min(rng.randint(1, 10), 1600000 // (c["n"] * c["K"])))
        c["R"], c["topk"], c["bounces"] = 128, rng.choice([256, 512]), rng.randint(3, 8)
    elif kind == "serve":
        c["n"] = _log(rng, 500, 20000)
        c["K"] = rng.choice([1, 4, 9, 16])
        c["lights"], c["R"], c["topk"], c["bounces"] = rng.randint(1, 4), 64, rng.choice([64, 128]), rng.randint(2, 8)
    elif kind == "dense":
        c["scene"] = "room"
        c["n"], c["R"], c["topk"], c["K"] = _log(rng, 2000, 32768), 256, 0, rng.choice([4, 9])
        c["lights"], c["bounces"] = _log(rng, 4, 100), rng.randint(3, 8)
    elif kind == "batch":
        many = rng.random() < 0.5
        c["scene"] = "room"
        c["rooms"], c["n_lo"], c["n_hi"] = rng.randint(4, 8), 2048, _log(rng, 4096, 12288)
        c["lights_lo"], c["lights_hi"] = (8, rng.randint(20, 100)) if many else (1, 4)
        c["R"], c["topk"], c["K"], c["bounces"] = 128, rng.choice([256, 512]), rng.choice([4, 9]), rng.randint(3, 8)
        c["bf16"] = rng.random() < 0.5
    elif kind == "hits":
        c["n"] = _log(rng, 3000, 40000)
        c["R"], c["topk"] = rng.choice([64, 100, 128]), rng.choice([0, 256, 512])
    elif kind == "sh":
        c["n"], c["R"], c["topk"] = _log(rng, 2000, 50000), 128, rng.choice([256, 512])
        c["K"], c["bounces"], c["lights"] = rng.choice([4, 9, 16]), rng.randint(3, 8), rng.choice([1, 1, 2])
        if c["lights"] == 2:
            c["n"] = min(c["n"], 20000)
    elif kind == "center":
        c["n"], c["R"], c["topk"] = _log(rng, 2000, 20000), 128, rng.choice([128, 256, 512])
    elif kind == "mc":
        c["n"], c["K"], c["lights"] = _log(rng, 4096, 50000), rng.choice([1, 4, 9]), rng.randint(1, 2)
        c["rounds"] = rng.randint(4, 16)
    else:
        c["n"], c["K"], c["lights"] = _log(rng, 4096, 32768), rng.choice([1, 4, 9, 16]), _log(rng, 1, 50)
    return c


# ---------------------------------------------------------------------------
# scenes
# ---------------------------------------------------------------------------
def _frames(nrm, rng):
    """Orthonormal tangents of unit normals, spun by a random angle, with
    t_u x t_v = n."""
    up = np.where(np.abs(nrm[:, :1]) < 0.9, np.array([[1.0, 0.0, 0.0]]), np.array([[0.0, 1.0, 0.0]]))
    a = np.cross(up, nrm)
    a /= np.linalg.norm(a, axis=1, keepdims=True)
    b = np.cross(nrm, a)
    ang = rng.uniform(0.0, 2.0 * math.pi, (nrm.shape[0], 1))
    return np.cos(ang) * a + np.sin(ang) * b, np.cos(ang) * b - np.sin(ang) * a


def _lattice(m, rng, jitter, lower=False):
    """A jittered spiral lattice on the unit sphere or its lower half."""
    k = np.arange(m) + 0.5
    y = -k / m if lower else 1.0 - 2.0 * k / m
    phi = np.arange(m) * (math.pi * (3.0 - math.sqrt(5.0))) + rng.uniform(0.0, 2.0 * math.pi)
    r = np.sqrt(np.maximum(0.0, 1.0 - y * y))
    p = np.stack([r * np.cos(phi), y, r * np.sin(phi)], 1) + rng.uniform(-jitter, jitter, (m, 3))
    p /= np.linalg.norm(p, axis=1, keepdims=True)
    if lower:
        p[:, 1] = -np.abs(p[:, 1])
    return p


def _spheres(rng, count, draw_radius, draw_center, fits):
    """Spheres that do not touch; fewer than `count` if they do not fit."""
    cs, rs = [], []
    for _ in range(20000):
        if len(cs) == count:
            break
        r = draw_radius()
        c = draw_center(r)
        if fits(c, r) and all(np.linalg.norm(c - c2) > r + r2 + 0.02 for c2, r2 in zip(cs, rs)):
            cs.append(c)
            rs.append(r)
    return cs, rs


def _pieces(n, areas):
    counts = np.floor(np.asarray(areas) / np.sum(areas) * n).astype(int)
    counts[0] += n - counts.sum()
    return counts


def _bowl(n, rng):
    """A hemispherical bowl of radius 1, front faces inwards, holding spheres."""
    cs, rs = _spheres(rng, 20, lambda: math.exp(rng.uniform(math.log(0.05), math.log(0.2))),
                      lambda r: rng.uniform(-1.0, 1.0, 3) * np.array([1.0, 0.5, 1.0]) - np.array([0.0, 0.5, 0.0]),
                      lambda c, r: np.linalg.norm(c) < 0.98 - r)
    areas = [2 * math.pi] + [4 * math.pi * r * r for r in rs]
    counts, h = _pieces(n, areas), math.sqrt(sum(areas) / n)
    q = _lattice(counts[0], rng, 0.25 * h, lower=True)
    P, N = [q], [-q]
    for c, r, m in zip(cs, rs, counts[1:]):
        q = _lattice(int(m), rng, 0.25 * h / r)
        P.append(c + r * q)
        N.append(q)
    return np.concatenate(P), np.concatenate(N), h, rng.beta(8.0, 1.0, n), rng.uniform(0.1, 0.9, (n, 3))


def _room(n, rng):
    """Five walls of [-2, 2]^3, front faces inwards, around a few spheres."""
    cs, rs = _spheres(rng, int(rng.integers(2, 7)), lambda: rng.uniform(0.4, 1.0),
                      lambda r: rng.uniform(r - 1.95, 1.95 - r, 3), lambda c, r: True)
    areas = [80.0] + [4 * math.pi * r * r for r in rs]
    counts, h = _pieces(n, areas), math.sqrt(sum(areas) / n)
    m = int(counts[0])
    side = max(1, math.ceil(math.sqrt(m / 5)))
    cell = np.sort(rng.choice(5 * side * side, m, replace=False))
    wall, iu, iv = cell // (side * side), cell // side % side, cell % side
    uv = ((np.stack([iu, iv], 1) + 0.5 + rng.uniform(-0.25, 0.25, (m, 2))) / side - 0.5) * 4.0
    w = np.array([-2.0, 2.0, -2.0, 2.0, -2.0])[wall]          # y-, y+, x-, x+, z-
    axis = np.array([1, 1, 0, 0, 2])[wall]
    P0, N0, i = np.empty((m, 3)), np.zeros((m, 3)), np.arange(m)
    P0[i, axis], P0[i, (axis + 1) % 3], P0[i, (axis + 2) % 3] = w, uv[:, 0], uv[:, 1]
    N0[i, axis] = -np.sign(w)
    P, N = [P0], [N0]
    for c, r, k in zip(cs, rs, counts[1:]):
        q = _lattice(int(k), rng, 0.25 * h / r)
        P.append(c + r * q)
        N.append(q)
    return np.concatenate(P), np.concatenate(N), h, rng.uniform(0.85, 1.0, n), rng.uniform(0.2, 0.8, (n, 3))


def _sphere(n, rng):
    """Inward surfels on the unit sphere."""
    q = rng.standard_normal((n, 3))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    return q, -q, 0.08 * math.sqrt(512.0 / n), np.full(n, 0.99), np.full((n, 3), 0.5)


_SCENES = {"bowl": _bowl, "room": _room, "sphere": _sphere}


def _scene(kind, n, lights, seed):
    """(surfel fields, albedo, light positions, light intensities) on the GPU."""
    rng = np.random.default_rng(seed)
    P, N, h, op, alb = _SCENES[kind](n, rng)
    tu, tv = _frames(N, rng)
    cols = [P[:, 0], P[:, 1], P[:, 2], tu[:, 0], tu[:, 1], tu[:, 2], tv[:, 0], tv[:, 1], tv[:, 2],
            N[:, 0], N[:, 1], N[:, 2], np.full(n, h), np.full(n, h), op]
    sur = {f: torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for f, v in zip(FIELDS, cols)}
    if kind == "bowl":
        lp = np.array([0.0, 1.4, 0.0]) + rng.uniform(-0.4, 0.4, (lights, 3))
    elif kind == "room":
        lp = rng.uniform(-1.8, 1.8, (lights, 3))
    else:
        lp = rng.uniform(-0.1, 0.1, (lights, 3))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()  # noqa: E731
    return sur, dev(alb), dev(lp), torch.full((lights,), 4.0, device="cuda")


def _uniform(shape, seed, lo=0.0, hi=1.0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(shape, generator=gen, device="cuda") * (hi - lo) + lo


def _rooms(c):
    """(surfels, lights) of every room of a batch: log-uniform sizes, the
    smallest and the largest of the range among them."""
    rng = np.random.default_rng(c["rooms"] + c["n_hi"])
    n = [int(round(math.exp(rng.uniform(math.log(c["n_lo"]), math.log(c["n_hi"]))))) for _ in range(c["rooms"])]
    n[0], n[-1] = c["n_lo"], c["n_hi"]
    return n, [int(rng.integers(c["lights_lo"], c["lights_hi"] + 1)) for _ in n]


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
# How many entries F has depends on the seed, so what has one value per entry
# is handed out in a buffer of the most entries such an F can have.
def _most(c, n):
    return n * min(n, c["topk"] if c["topk"] else 20 * c["R"])


def _whole(x, most):
    out = torch.zeros(most, dtype=x.dtype, device="cuda")
    out[:x.shape[0]] = x
    return out


def _csr(ff, most):
    rp, col, val = ff.csr()
    return rp, _whole(col, most), _whole(val, most)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": case, "seed": seed, "ff": None, "bvh": None, "tape": None}
    if kind == "batch":
        n, lights = _rooms(c)
        s["ffs"], s["rooms"] = [], n
        for k, m in enumerate(n):
            bvh = g.build_bvh(_scene(c["scene"], m, 1, seed * 64 + k)[0])
            s["ffs"].append(g.form_factors(bvh, c["R"], seed + k, t_min=T_MIN, topk=c["topk"], records=False,
                                           compact=True))
        s["batch"] = g.batch_create(s["ffs"], lights, c["K"])
        if c["bf16"]:
            g.batch_set_precision(s["batch"], g.BF16)
        vals = sum(m * lt * c["K"] * 3 for m, lt in zip(n, lights))
        s["rho"] = _uniform((sum(n), 3), seed, 0.2, 0.8)
        s["E"], s["gB"] = _uniform(vals, seed + 1), _uniform(vals, seed + 2, -1e-3, 1e-3)
        s["B"], s["gE"] = torch.empty_like(s["E"]), torch.empty_like(s["E"])
        return s
    n, lights, K = c["n"], c.get("lights", 1), c.get("K", 1)
    s["sur"], s["alb"], s["lp"], s["lI"] = _scene(c["scene"], n, lights, seed)
    s["gB"] = _uniform((n, lights, K, 3), seed + 2, -1e-3, 1e-3)
    if kind == "step":
        return s
    s["bvh"] = g.build_bvh(s["sur"])
    s["rho"] = g.reflectance(s["bvh"], s["alb"])
    if kind in ("fixed", "serve", "dense", "hits", "sh", "center"):
        s["ff"] = g.form_factors(s["bvh"], c["R"], seed, t_min=T_MIN, topk=c["topk"], records=kind == "hits",
                                 compact=kind != "hits")
    if kind in ("fixed", "serve", "dense", "sh"):
        s["E"] = _uniform((n, lights, K, 3), seed + 1)
        s["B"] = torch.empty_like(s["E"])
    if kind == "dense":
        g.ff_dense(s["ff"])
    elif kind == "hits":
        s["gF"] = _uniform(s["ff"].info()[1], seed + 3, -1.0, 1.0)
        s["grho"] = _uniform((n, 3), seed + 4, -1.0, 1.0)
    elif kind == "sh":
        s["mat"] = (_uniform(n, seed + 3), _uniform((n, 3), seed + 4, 0.1, 0.9), _uniform((n, 3), seed + 5, 0.1, 0.9),
                    _uniform(n, seed + 6, 1.0, 20.0))
        s["Rm"] = g.brdf_reflectance(s["bvh"], *s["mat"], K)
    elif kind == "center":
        s["lam"] = _uniform(n, seed + 3, 0.2, 0.8)
        s["gF"] = _uniform(s["ff"].info()[1], seed + 4, -1.0, 1.0)
        s["fc"] = g.ff_center(s["bvh"], s["ff"], s["lam"])
    elif kind == "mc":
        s["lam"] = torch.full((n,), 0.5, device="cuda")
        s["E"] = g.direct_light(s["bvh"], s["alb"], s["lp"], s["lI"], K)
        s["mc"] = g.mc_create(s["bvh"])
    elif kind == "lights":
        s["E"] = torch.empty_like(s["gB"])
    return s


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    most = sum(_most(c, m) for m in s["rooms"]) if kind == "batch" else _most(c, c["n"]) if "topk" in c else 0
    if kind == "step":
        bvh = s["bvh"] = g.build_bvh(s["sur"], s["bvh"])
        ff = s["ff"] = g.form_factors(bvh, c["R"], s["seed"], t_min=T_MIN, topk=c["topk"], ff=s["ff"])
        E = g.direct_light(bvh, s["alb"], s["lp"], s["lI"], c["K"])
        if c["autograd"]:
            op, alb, E = s["sur"]["opacity"].clone().requires_grad_(), s["alb"].clone().requires_grad_(), E.requires_grad_()
            B = g.RadiosityFn.apply(op, alb, E, bvh, ff, c["bounces"])
            B.backward(s["gB"])
            return {"F": _csr(ff, most), "E": E.detach(), "B": B.detach(), "gE": E.grad, "go": op.grad, "ga": alb.grad}
        rho = g.reflectance(bvh, s["alb"])
        B, s["tape"] = g.transport_solve(ff, rho, E, c["bounces"], tape=s["tape"])
        gE, grho, gF = g.transport_backward(ff, s["tape"], rho, s["gB"])
        go, ga = g.opacity_backward(bvh, ff, gF, grho, s["alb"])
        return {"F": _csr(ff, most), "E": E, "B": B, "gE": gE, "grho": grho, "gF": _whole(gF, most), "go": go, "ga": ga}
    if kind in ("fixed", "dense"):
        B, s["tape"] = g.transport_solve(s["ff"], s["rho"], s["E"], c["bounces"], tape=s["tape"], out=s["B"],
                                         precision=g.BF16 if kind == "dense" else g.FP32)
        gE, grho, gF = g.transport_backward(s["ff"], s["tape"], s["rho"], s["gB"])
        return {"B": B, "gE": gE, "grho": grho, "gF": _whole(gF, most)}
    if kind == "serve":
        return {"B": g.transport_solve_noalloc(s["ff"], s["rho"], s["E"], c["bounces"], s["B"])}
    if kind == "batch":
        B = g.batch_transport_solve(s["batch"], s["rho"], s["E"], c["bounces"], out=s["B"])
        gE, grho, gF = g.batch_transport_backward(s["batch"], s["rho"], s["gB"], out=s["gE"])
        return {"B": B, "gE": gE, "grho": grho, "gF": _whole(gF, most)}
    if kind == "hits":
        go, ga = g.opacity_backward(s["bvh"], s["ff"], s["gF"], s["grho"], s["alb"])
        return {"go": go, "ga": ga, "geometry": g.geometry_backward(s["bvh"], s["ff"], s["gF"])}
    if kind == "sh":
        B, s["tape"] = g.transport_solve_sh(s["ff"], s["bvh"], s["Rm"], s["E"], c["bounces"], tape=s["tape"],
                                            out=s["B"])
        gE, gR, gF = g.transport_backward_sh(s["ff"], s["bvh"], s["tape"], s["Rm"], s["gB"])
        return {"B": B, "gE": gE, "gR": gR, "gF": _whole(gF, most), "materials": g.brdf_backward(s["bvh"], *s["mat"], gR)}
    if kind == "center":
        fc = s["fc"] = g.ff_center(s["bvh"], s["ff"], s["lam"], ff=s["fc"])
        gl, geo = g.ff_center_backward(s["bvh"], fc, s["lam"], s["gF"])
        return {"F": _csr(fc, most), "glam": gl, "geometry": geo}
    if kind == "mc":
        B, visits = g.mc_solve(s["mc"], s["lam"], s["rho"], s["E"], c["rounds"], s["seed"])
        return {"B": B, "visits": visits}
    E = g.direct_light(s["bvh"], s["alb"], s["lp"], s["lI"], c["K"], out=s["E"])
    glp, glI, ga, geo = g.direct_light_backward(s["bvh"], s["alb"], s["lp"], s["lI"], s["gB"])
    return {"E": E, "glp": glp, "glI": glI, "ga": ga, "geometry": geo}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _entries(c, n):
    """Stored entries of a ray-cast F: a row of these scenes has about 15
    distinct senders a ray, in a small scene a third of all surfels at most."""
    full = min(0.33 * n, 14.7 * c["R"])
    return n * (min(c["topk"], full) if c["topk"] else full)


def work(case):
    c, kind = case, case["kind"]
    if kind == "batch":
        n, lights = _rooms(c)
        nnz = [_entries(c, m) for m in n]
        cols = [lt * c["K"] * 3 for lt in lights]
        vals = sum(m * x for m, x in zip(n, cols))
        return {"bytes": 16.0 * vals + 12.0 * sum(nnz) + 24.0 * sum(n),
                "flops": sum(6.0 * c["bounces"] * z * x for z, x in zip(nnz, cols))}
    n, lights, K = c["n"], c.get("lights", 1), c.get("K", 1)
    cols, depth = lights * K * 3, math.log2(n)
    ray = 2 * depth * 24 + 28 * 70                       # boxes on the way and some 28 composited hits
    segment = 2 * depth * 24 + 10 * 40
    if kind in ("step", "fixed", "sh", "serve", "dense"):
        nnz = _entries(c, n)
        per = 2.0 * (K * 2 if kind == "sh" else 1) * nnz * cols
        if kind == "serve":
            return {"bytes": 8.0 * nnz + 8.0 * n * cols + 12 * n, "flops": c["bounces"] * per}
        if kind == "dense":
            per = 2.0 * n * n * cols
        w = {"bytes": 12.0 * nnz + 16.0 * n * cols + 24 * n, "flops": 3.0 * c["bounces"] * per}
        if kind == "step":
            w["bytes"] += 8.0 * nnz + 100.0 * n
            w["flops"] += n * c["R"] * ray * 1.5 + n * lights * segment
        return w
    if kind == "hits":
        hits = n * c["R"] * 28.0
        return {"bytes": 8.0 * hits + 8.0 * _entries(c, n) + 140.0 * n, "flops": hits * 120}
    if kind == "center":
        nnz = _entries(c, n)
        return {"bytes": 16.0 * nnz + 130.0 * n, "flops": 2 * nnz * segment}
    if kind == "mc":
        return {"bytes": 12.0 * n * cols + 100.0 * n, "flops": c["rounds"] * n * (2 * math.sqrt(n) * 30 + segment)}
    return {"bytes": 8.0 * n * cols + 160.0 * n, "flops": 3.0 * n * lights * segment}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
# F is an input of the transport: where a pass starts from an F in hand, that
# F's stored entries are taken as they are; hit lists have no 64-bit value.
def _blocks(csr, n, transpose=False, step=4096):
    """(first row, rows as a dense FP64 matrix) of F, or of F^T."""
    rp, col, val = csr
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rp.diff())
    col, val = col.long(), val.double()
    if transpose:
        order = torch.argsort(col, stable=True)
        rows, col, val = col[order], rows[order], val[order]
        rp = torch.zeros(n + 1, dtype=torch.long, device="cuda")
        rp[1:] = torch.bincount(rows, minlength=n).cumsum(0)
    for a in range(0, n, step):
        b = min(n, a + step)
        x, y = int(rp[a]), int(rp[b])
        D = torch.zeros((b - a, n), dtype=torch.float64, device="cuda")
        D[rows[x:y] - a, col[x:y]] = val[x:y]
        yield a, D


def _times(csr, n, transpose=False):
    """x -> F x (or F^T x) for x [n, C]; the dense blocks are kept while they are few."""
    kept = list(_blocks(csr, n, transpose)) if n <= 40000 else None

    def f(x):
        out = torch.empty_like(x)
        for a, D in kept if kept is not None else _blocks(csr, n, transpose):
            out[a:a + D.shape[0]] = D @ x
        return out
    return f


def _transport(csr, rho, E, gB, nb, backward=True):
    """B, and the adjoint's dL/dE, dL/drho, dL/dF of E, gB [n, C]."""
    n, C = E.shape
    r = rho.double().repeat(1, C // 3)
    E, gB = E.double(), gB.double()
    F = _times(csr, n)
    tape = [E]
    for _ in range(nb):
        tape.append(E + r * F(tape[-1]))
    if not backward:
        return tape[-1]
    Ft = _times(csr, n, transpose=True)
    lam, gE = [gB], gB.clone()
    for _ in range(nb):
        lam.append(Ft(r * lam[-1]))
        gE += lam[-1]
    rp, col, val = csr
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rp.diff())
    gF = torch.empty(col.shape[0], dtype=torch.float64, device="cuda")
    grho = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    if C > 600 and n > 1000:                              # every pair by dense products, then the stored ones
        a = torch.cat([lam[nb - 1 - k].view(n, -1, 3) for k in range(nb)], 1)
        b = torch.cat([tape[k].view(n, -1, 3) for k in range(nb)], 1)
        S = [a[:, :, q].contiguous() for q in range(3)], [b[:, :, q].t().contiguous() for q in range(3)]
        del a, b
        step = 4096
        for i in range(0, n, step):
            x, y = int(rp[i]), int(rp[min(n, i + step)])
            at, to = rows[x:y], col[x:y].long()
            s = torch.stack([(S[0][q][i:i + step] @ S[1][q])[at - i, to] for q in range(3)], 1)
            gF[x:y] = (s * rho.double()[at]).sum(1)
            grho.index_add_(0, at, s * val[x:y].double()[:, None])
    else:
        step = max(1, (1 << 26) // C)
        for x in range(0, col.shape[0], step):
            at, to = rows[x:x + step], col[x:x + step].long()
            s = 0.0
            for k in range(nb):
                s = s + (lam[nb - 1 - k][at] * tape[k][to]).view(at.shape[0], -1, 3).sum(1)
            gF[x:x + step] = (s * rho.double()[at]).sum(1)
            grho.index_add_(0, at, s * val[x:x + step].double()[:, None])
    return tape[-1], gE, grho, gF


def _direct(sur, alb, lp, lI, K):
    """Point lights through all surfels on the way: E [n, Lt, K, 3]."""
    d = {f: v.double() for f, v in sur.items()}
    p, tu, tv, nr = (torch.stack([d[a + x] for x in "xyz"], 1) for a in ("p", "tu", "tv", "n"))
    op = d["opacity"].clamp(0.0, 0.9999)
    dens = -torch.log1p(-op)
    n, lp = p.shape[0], lp.double()
    box = (p.max(0).values - p.min(0).values)
    eps = 1e-5 * float(box.norm())
    own = [(p * a).sum(1) for a in (nr, tu, tv)]
    E = torch.zeros((n, lp.shape[0], K, 3), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 24) // n)
    for i in range(0, n, step):
        q = p[i:i + step]
        dn, du, dv = (o[None] - q @ a.t() for o, a in zip(own, (nr, tu, tv)))   # (p_j - p_i) in j's frame
        me = torch.arange(i, i + q.shape[0], device="cuda")
        for k in range(lp.shape[0]):
            w = lp[k] - q
            r = w.norm(dim=1)
            cos = (w * nr[i:i + step]).sum(1) / r
            den = w @ nr.t()
            t = dn / den
            u = (t * (w @ tu.t()) - du) / d["su"]
            v = (t * (w @ tv.t()) - dv) / d["sv"]
            r2 = u * u + v * v
            hit = (den.abs() > 1e-6) & (t > eps / r[:, None]) & (t < 1.0) & (r2 <= 9.0)
            hit[torch.arange(q.shape[0], device="cuda"), me] = False
            T = torch.exp(-torch.where(hit, dens * torch.exp(-1.7 * r2), 0.0).sum(1))
            base = op[i:i + step] * (2.0 / math.sqrt(math.pi)) * lI[k].double() * cos.clamp(min=0.0) / r ** 2 * T
            E[i:i + step, k, 0] = base[:, None] * alb[i:i + step].double()
    return E


def _sh(w, K):
    """Real spherical harmonics of unit vectors, degrees 0 to 3."""
    x, y, z = w.unbind(-1)
    s = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if K > 1:
        a = math.sqrt(0.75 / math.pi)
        s += [a * y, a * z, a * x]
    if K > 4:
        a = 0.5 * math.sqrt(15 / math.pi)
        s += [a * x * y, a * y * z, 0.25 * math.sqrt(5 / math.pi) * (3 * z * z - 1), a * x * z, 0.5 * a * (x * x - y * y)]
    if K > 9:
        a, b = 0.25 * math.sqrt(17.5 / math.pi), 0.25 * math.sqrt(10.5 / math.pi)
        e = 0.5 * math.sqrt(105 / math.pi)
        s += [a * y * (3 * x * x - y * y), e * x * y * z, b * y * (5 * z * z - 1),
              0.25 * math.sqrt(7 / math.pi) * z * (5 * z * z - 3), b * x * (5 * z * z - 1),
              0.5 * e * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(s, -1)


def _transport_sh(csr, sur, Rm, E, gB, nb):
    n, Lt, K, _ = E.shape
    d = {f: v.double() for f, v in sur.items()}
    p = torch.stack([d["p" + x] for x in "xyz"], 1)
    frame = torch.stack([torch.stack([d[a + x] for x in "xyz"], 1) for a in ("tu", "tv", "n")], 1)   # [n, 3, xyz]
    rp, col, val = csr
    rows, col, val = torch.repeat_interleave(torch.arange(n, device="cuda"), rp.diff()), col.long(), val.double()
    Rm, E, gB = Rm.double()[:, None], E.double(), gB.double()
    step = 1 << 20

    def pairs(x):
        i, j = rows[x:x + step], col[x:x + step]
        w = p[j] - p[i]
        w = w / w.norm(dim=1, keepdim=True)
        Yi = _sh((frame[i] * w[:, None]).sum(2), K)
        Yj = _sh(-(frame[j] * w[:, None]).sum(2), K)
        return i, j, val[x:x + step], Yi, Yj

    def move(X, back=False):
        out = torch.zeros_like(X)
        for x in range(0, col.shape[0], step):
            i, j, f, Yi, Yj = pairs(x)
            if back:
                i, j, Yi, Yj = j, i, Yj, Yi
            m = (X[j] * Yj[:, None, :, None]).sum(2) * f[:, None, None]
            out.index_add_(0, i, m[:, :, None, :] * Yi[:, None, :, None])
        return out

    tape, moved = [E], []
    for _ in range(nb):
        moved.append(move(tape[-1]))
        tape.append(E + Rm * moved[-1])
    lam, gE, gR = [gB], gB.clone(), torch.zeros_like(Rm)
    for k in range(nb - 1, -1, -1):
        gR += (lam[-1] * moved[k]).sum(1, keepdim=True)
        lam.append(move(Rm * lam[-1], back=True))
        gE += lam[-1]
    gF = torch.empty(col.shape[0], dtype=torch.float64, device="cuda")
    for x in range(0, col.shape[0], step):
        i, j, f, Yi, Yj = pairs(x)
        s = 0.0
        for k in range(nb):
            a = ((Rm * lam[nb - 1 - k])[i] * Yi[:, None, :, None]).sum(2)
            s = s + (a * (tape[k][j] * Yj[:, None, :, None]).sum(2)).sum((1, 2))
        gF[x:x + step] = s
    return tape[-1], gE, gR[:, 0], gF


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("hits", "center", "mc"):
        return None
    if kind in ("step", "lights"):
        # the traced outputs follow 32-bit hit decisions; direct light is a sum over all surfels
        if c["n"] ** 2 * c["lights"] > 3e10:
            return None
        sur, alb, lp, lI = _scene(c["scene"], c["n"], c["lights"], seed)
        E = _direct(sur, alb, lp, lI, c["K"])
        if kind == "lights":
            return {"E": E, "glp": None, "glI": None, "ga": None, "geometry": None}
        r = {"F": None, "E": E, "B": None, "gE": None, "go": None, "ga": None}
        return r if c["autograd"] else {**r, "grho": None, "gF": None}
    s = prepare(case, seed)
    nb = c["bounces"]
    if kind == "batch":
        n, lights = _rooms(c)
        out, at, row = [], 0, 0
        for ff, m, lt in zip(s["ffs"], n, lights):
            C = lt * c["K"] * 3
            E, gB = (s[k][at:at + m * C].view(m, C) for k in ("E", "gB"))
            out.append(_transport(ff.csr(), s["rho"][row:row + m], E, gB, nb))
            at, row = at + m * C, row + m
        B, gE, grho, gF = zip(*out)
        return {"B": torch.cat([b.reshape(-1) for b in B]), "gE": torch.cat([b.reshape(-1) for b in gE]),
                "grho": torch.cat(grho), "gF": _whole(torch.cat(gF), sum(_most(c, m) for m in n))}
    csr, shape = s["ff"].csr(), s["E"].shape
    if kind == "sh":
        B, gE, gR, gF = _transport_sh(csr, s["sur"], s["Rm"], s["E"], s["gB"], nb)
        return {"B": B, "gE": gE, "gR": gR, "gF": _whole(gF, _most(c, c["n"])), "materials": None}
    E, gB = s["E"].reshape(shape[0], -1), s["gB"].reshape(shape[0], -1)
    if kind == "serve":
        return {"B": _transport(csr, s["rho"], E, gB, nb, backward=False).view(shape)}
    s["ff"] = None
    B, gE, grho, gF = _transport(csr, s["rho"], E, gB, nb)
    return {"B": B.view(shape), "gE": gE.view(shape), "grho": grho, "gF": _whole(gF, _most(c, c["n"]))}
