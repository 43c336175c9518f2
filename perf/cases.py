"""The work whose speed matters: calls of the public API on synthetic clouds.

Every case is one pass of something a program does with this framework,
through `paper_1902_01061_amd`: whole registrations of a small pair, a
scan, a depth-frame scene, a batch and a multi-start sweep; the single calls
they are made of (descriptors, one step, the force field and its gradient,
vector descriptors); and what follows a registration (residual, change
detection).  `exact` evaluates the same results in float64 with plain torch
and numpy, from the method's equations.

Clouds are drawn on the GPU from the seed: an ellipsoid fused with a planar
patch (small pairs, batches), a bumpy closed surface with a missing cap,
blob and uniform outliers (scans) and a depth frame of a room with boxes
(scenes); both clouds of a pair carry sensor noise.
"""
import math
import os

import numpy as np
import torch

import paper_1902_01061_amd as sg

DEV = "cuda"
F64 = torch.float64
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES = os.path.join(ROOT, "paper_1902_01061_amd", "tiles_gfx950.json")
G1 = 10000.0
SUMS = 8  # flags bit 3: pair sums of the p = 1 law formed once per registration

_CTX = None


def _ctx():
    """The program's one context, with the committed launch shapes loaded."""
    global _CTX
    if _CTX is None:
        _CTX = sg.Context(0)
        if os.path.exists(TILES):
            _CTX.load_tiles(TILES)
    return _CTX


# ------------------------------------------------------------------- cases
def listed():
    return [
        # a small pair registered from scratch (an object model against a
        # segmented view): 100 short iterations, where latency counts
        {"name": "register_small", "kind": "register", "cloud": "surface", "m": 1024, "n": 1024, "k": 16, "p": 1.0,
         "g_mode": 0, "flags": 0, "E": 100},
        # two laser scans, the everyday registration of the p = 1 law: pair
        # sums once, then 300 cheap iterations
        {"name": "register_scan_sums", "kind": "register", "cloud": "scan", "m": 32400, "n": 36000, "k": 24, "p": 1.0,
         "g_mode": 0, "flags": SUMS, "E": 300},
        # two depth frames, all pairs evaluated in every iteration: the
        # largest single registration (20 iterations: where the paper's
        # example reaches its minimum)
        {"name": "register_scene", "kind": "register", "cloud": "scene", "m": 250000, "n": 307200, "k": 16, "p": 1.0,
         "g_mode": 1, "flags": 0, "E": 20},
        # uneven pairs registered in one call (parts of an assembly)
        {"name": "batch_sums", "kind": "batch", "B": 48, "nmin": 2000, "nmax": 40000, "k": 16, "flags": SUMS,
         "E": 100},
        # initial rotations tried for one pair whose pose is unknown
        {"name": "multistart_sums", "kind": "multistart", "S": 32, "m": 22000, "n": 20000, "k": 16, "flags": SUMS,
         "E": 100},
        # one iteration of the d^2 law with its wrench and per-point forces
        # (a program that runs its own loop)
        {"name": "step_scan", "kind": "step", "m": 32400, "n": 36000, "p": 2.0, "g_mode": 0, "flags": 0,
         "masses": False},
        # descriptors of one depth frame as it arrives
        {"name": "descriptors_scene", "kind": "descriptors", "cloud": "scene", "n": 307200, "k": 16},
        # vector descriptors of two scans and one step with them
        {"name": "vector_scan", "kind": "vector", "m": 32400, "n": 36000, "k": 24, "D": 16},
        # what changed between two registered depth frames
        {"name": "change_scene", "kind": "change", "m": 250000, "n": 307200, "k": 16, "tau": 0.05},
        # how well a scan is registered
        {"name": "residual_scan", "kind": "residual", "cloud": "scan", "m": 32400, "n": 36000},
        # force field and its gradient inside a training step
        {"name": "force_grad", "kind": "force_grad", "m": 8192, "n": 8192, "p": 2.0},
        # 50 unrolled iterations differentiated with respect to the
        # bandwidths and the initial pose
        {"name": "unrolled", "kind": "unrolled", "m": 8192, "n": 8192, "E": 50, "K": 10},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["register_small", "register_sums", "register_scene", "batch", "multistart", "step",
                       "descriptors", "vector", "change", "residual", "force_grad", "unrolled"])
    if kind == "register_small":
        n = _log_int(rng, 200, 6000)
        return {"kind": "register", "cloud": "surface", "m": max(100, int(n * rng.uniform(0.7, 1.3))), "n": n,
                "k": rng.choice([8, 16, 24]), "p": 1.0, "g_mode": rng.choice([0, 1]), "flags": 0,
                "E": rng.randint(20, 150)}
    if kind == "register_sums":
        n = _log_int(rng, 2000, 120000)
        return {"kind": "register", "cloud": "scan", "m": int(n * 0.9), "n": n, "k": rng.choice([8, 16, 24, 32]),
                "p": 1.0, "g_mode": rng.choice([0, 1]), "flags": SUMS, "E": rng.randint(20, 300)}
    if kind == "register_scene":
        n = _log_int(rng, 20000, 307200)
        return {"kind": "register", "cloud": "scene", "m": int(n * rng.uniform(0.5, 0.81)), "n": n, "k": 16, "p": 1.0,
                "g_mode": rng.choice([0, 1]), "flags": 0, "E": rng.randint(5, 20)}
    if kind == "batch":
        nmin = _log_int(rng, 500, 4000)
        return {"kind": "batch", "B": rng.randint(3, 48), "nmin": nmin, "nmax": nmin * rng.randint(2, 10),
                "k": rng.choice([8, 16, 24]), "flags": SUMS, "E": rng.randint(20, 100)}
    if kind == "multistart":
        n = _log_int(rng, 1000, 20000)
        return {"kind": "multistart", "S": rng.randint(4, 32), "m": int(n * rng.uniform(0.8, 1.1)), "n": n, "k": 16,
                "flags": SUMS, "E": rng.randint(20, 100)}
    if kind == "step":
        n = _log_int(rng, 500, 60000)
        p = rng.choice([1.0, 2.0, 3.0, -2.0])  # -2: the softened inverse-square law, masses alone
        return {"kind": "step", "m": int(n * 0.9), "n": n, "p": p, "g_mode": 2 if p < 0 else rng.choice([0, 1]),
                "flags": rng.choice([0, 2]) if p == 1.0 else 0, "masses": rng.random() < 0.5}
    if kind == "descriptors":
        return {"kind": "descriptors", "cloud": rng.choice(["scan", "scene", "surface"]),
                "n": _log_int(rng, 500, 307200), "k": rng.choice([8, 16, 24, 32])}
    if kind == "vector":
        n = _log_int(rng, 1000, 40000)
        return {"kind": "vector", "m": int(n * 0.9), "n": n, "k": rng.choice([16, 24]), "D": rng.choice([8, 12, 16])}
    if kind == "change":
        n = _log_int(rng, 5000, 307200)
        return {"kind": "change", "m": int(n * rng.uniform(0.5, 0.81)), "n": n, "k": 16,
                "tau": round(rng.uniform(0.02, 0.1), 4)}
    if kind == "residual":
        n = _log_int(rng, 1000, 200000)
        return {"kind": "residual", "cloud": rng.choice(["scan", "surface"]), "m": int(n * 0.9), "n": n}
    n = _log_int(rng, 500, 12000 if kind == "force_grad" else 8192)
    m = int(n * rng.uniform(0.7, 1.0))
    if kind == "force_grad":
        return {"kind": "force_grad", "m": m, "n": n, "p": rng.choice([1.0, 2.0])}
    return {"kind": "unrolled", "m": m, "n": n, "E": rng.randint(10, 50), "K": 10}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (int(seed) + 1))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=F64)


def _unit(g, n):
    u = _randn(g, n, 3)
    return u / u.norm(dim=1, keepdim=True)


def _rotation(g, lo_deg, hi_deg):
    a = _unit(g, 1)[0]
    th = math.radians(lo_deg + (hi_deg - lo_deg) * float(_rand(g, 1)))
    x, y, z = (float(v) for v in a)
    K = torch.tensor([[0, -z, y], [z, 0, -x], [-y, x, 0]], device=DEV, dtype=F64)
    return torch.eye(3, device=DEV, dtype=F64) + math.sin(th) * K + (1 - math.cos(th)) * (K @ K)


def _surface(g, n):
    """Ellipsoid (1, 0.6, 0.4) fused with a 1.0 x 0.8 patch, uniform by area."""
    a, b, c = 1.0, 0.6, 0.4
    pp = 1.6075
    area = 4 * math.pi * (((a * b) ** pp + (a * c) ** pp + (b * c) ** pp) / 3) ** (1 / pp)
    n_e = int(round(n * area / (area + 0.8)))
    u = _unit(g, 3 * n_e + 256)
    w = ((b * c * u[:, 0]) ** 2 + (a * c * u[:, 1]) ** 2 + (a * b * u[:, 2]) ** 2).sqrt()
    u = u[_rand(g, len(u)) * max(b * c, a * c, a * b) < w][:n_e]
    patch = _rand(g, n - len(u), 3) - 0.5
    patch[:, 1] *= 0.8
    patch[:, 2] = -c
    return torch.cat([u * torch.tensor([a, b, c], device=DEV, dtype=F64), patch])


def _bumpy(g, n):
    """Closed radial surface with smooth random bumps."""
    u = _unit(g, n)
    r = torch.ones(n, device=DEV, dtype=F64)
    for q in range(1, 7):
        d, ph = _unit(g, 6) * q, _rand(g, 6) * 2 * math.pi
        r = r + (0.06 / q * torch.cos(u @ d.T + ph)).sum(1)
    return u * r.clamp(min=0.5)[:, None]


def _room(g, n, boxes, R, sd=0.001):
    """n pixels of a depth frame of a 5 x 3 x 4 m room seen from the origin."""
    h = max(8, int(math.ceil(math.sqrt(n * 0.75))))
    w = -(-n // h)
    f = 525.0 * w / 640.0
    v, u = torch.meshgrid(torch.arange(h, device=DEV, dtype=F64), torch.arange(w, device=DEV, dtype=F64),
                          indexing="ij")
    d = torch.stack([(u - (w - 1) / 2) / f, -(v - (h - 1) / 2) / f, torch.ones_like(u)], -1).reshape(-1, 3)
    if h * w > n:
        d = d[torch.randperm(h * w, generator=g, device=DEV)[:n].sort().values]
    inv = 1.0 / (d @ R.T)
    lo = torch.tensor([-2.5, -1.2, -0.5], device=DEV, dtype=F64)
    hi = torch.tensor([2.5, 1.8, 3.5], device=DEV, dtype=F64)
    z = torch.maximum(lo * inv, hi * inv).amin(1)
    for b in boxes:
        t0, t1 = b[0] * inv, b[1] * inv
        near, far = torch.minimum(t0, t1).amax(1), torch.maximum(t0, t1).amin(1)
        z = torch.where((far >= near) & (near > 1e-6) & (near < z), near, z)
    return d * (z + _randn(g, len(d)) * sd * z * z)[:, None]


def _scene_pair(g, m, n):
    """A room of 20 boxes, and the room with one box removed and two added
    seen from a camera turned by 30 degrees; y = R x."""
    s = 0.2 + 0.6 * _rand(g, 22, 3)
    c = torch.stack([-2 + 4 * _rand(g, 22), 0.8 + 2.2 * _rand(g, 22)], 1)
    lo = torch.stack([c[:, 0] - s[:, 0] / 2, torch.full((22,), -1.2, device=DEV, dtype=F64), c[:, 1] - s[:, 2] / 2], 1)
    boxes = list(torch.stack([lo, lo + s], 1))
    p, y = math.radians(20.0), math.radians(30.0)
    pitch = torch.tensor([[1, 0, 0], [0, math.cos(p), -math.sin(p)], [0, math.sin(p), math.cos(p)]], device=DEV,
                         dtype=F64)
    yaw = torch.tensor([[math.cos(y), 0, math.sin(y)], [0, 1, 0], [-math.sin(y), 0, math.cos(y)]], device=DEV,
                       dtype=F64)
    X = _room(g, n, boxes[:20], pitch)
    Y = _room(g, m, boxes[1:], yaw @ pitch)
    return X, Y, (1.0, (yaw @ pitch).T @ pitch, torch.zeros(3, device=DEV, dtype=F64))


def _scan_pair(g, m, n):
    """A scan and a second one with a missing cap, a blob and uniform
    outliers, turned by 60 degrees and scaled."""
    base = _bumpy(g, n)
    X = base + 0.003 * _randn(g, n, 3)
    kept = max(1, int(m / 1.2))
    v = _unit(g, 1)[0]
    order = ((base / base.norm(dim=1, keepdim=True)) @ v).argsort()
    keep = base[order[: max(kept, int(0.75 * n))]]
    keep = keep[torch.randperm(len(keep), generator=g, device=DEV)[:kept]]
    nb = int(0.15 * len(keep))
    blob = 0.8 * _unit(g, 1) + 0.1 * _randn(g, nb, 3)
    lo, hi = base.amin(0), base.amax(0)
    uni = lo + (hi - lo) * _rand(g, m - len(keep) - nb, 3)
    s, R, t = 0.8, _rotation(g, 60, 60), torch.zeros(3, device=DEV, dtype=F64)
    Y = s * (torch.cat([keep, blob, uni]) + 0.003 * _randn(g, m, 3)) @ R.T + t
    return X, Y, (s, R, t)


def _surface_pair(g, m, n, lo_deg=0.0, hi_deg=90.0):
    """An object and a noisy second view of it with 10 % uniform outliers
    under a random similarity transform."""
    base = _surface(g, n)
    X = base + 0.002 * _randn(g, n, 3)
    n_in = min(m, n)
    sel = base[torch.randperm(n, generator=g, device=DEV)[: min(n_in, int(m / 1.1) + 1)]]
    lo, hi = base.amin(0), base.amax(0)
    P = torch.cat([sel, lo + (hi - lo) * _rand(g, m - len(sel), 3)])
    s, R, t = 0.7 + 0.7 * float(_rand(g, 1)), _rotation(g, lo_deg, hi_deg), _rand(g, 3) - 0.5
    Y = s * P @ R.T + t + 0.005 * _randn(g, m, 3)
    return X, Y, (s, R, t)


PAIRS = {"surface": _surface_pair, "scan": _scan_pair, "scene": _scene_pair}


def _pair(case, seed):
    """(reference, template, transform) of a case as float32 (n, 3) tensors."""
    cloud = case.get("cloud") or {"step": "scan", "vector": "scan", "change": "scene", "multistart": "surface",
                                  "force_grad": "surface", "unrolled": "surface"}[case["kind"]]
    n = case["n"]
    X, Y, T = PAIRS[cloud](_gen(seed), case.get("m", n), n)
    return X.float(), Y.float(), T


def _batch_pairs(case, seed):
    g = _gen(seed)
    r = np.random.RandomState(seed % (1 << 31))
    out = []
    for _ in range(case["B"]):
        n = int(round(math.exp(r.uniform(math.log(case["nmin"]), math.log(case["nmax"])))))
        X, Y, _ = _surface_pair(g, int(1.1 * n), n)
        out.append((X.float(), Y.float()))
    return out


def _inverse_pose(T, g):
    """The pose that undoes T, a little off as after a registration."""
    s, R, t = T
    Ri = R.T @ _rotation(g, 0.2, 0.4)
    off = 0.005 * _randn(g, 3)
    return torch.cat([torch.tensor([1.0 / s], device=DEV, dtype=F64), Ri.reshape(-1), off - Ri @ t / s])


def _rotations(S):
    """S well-spread rotations (quaternions along a spiral)."""
    out = np.empty((S, 3, 3))
    for i in range(S):
        s = i + 0.5
        r, q = math.sqrt(s / S), math.sqrt(1.0 - s / S)
        al, be = 2 * math.pi * s / math.sqrt(2.0), 2 * math.pi * s / 1.533751168755204288118041
        w, x, y, z = r * math.sin(al), r * math.cos(al), q * math.sin(be), q * math.cos(be)
        out[i] = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                  [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                  [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    return out


def _params(case, **kw):
    return sg.Params(**{q: case[q] for q in ("p", "g_mode", "k", "flags", "E") if q in case}, **kw)


def _masses(case, seed):
    """Reference and template masses (or None, None) of a step."""
    if not case.get("masses"):
        return None, None
    g = _gen(seed + 15485863)
    return (0.5 + 1.5 * _rand(g, case["n"])).float(), (0.5 + 1.5 * _rand(g, case["m"])).float()


def _soft(case, X):
    """Softening of a step: 5 % of the length scale for the inverse-square law."""
    return 0.05 * math.sqrt(_moments(X)[2]) if case["p"] < 1.0 else 0.0


def _grads_in(case, seed):
    """Upstream gradients of the training steps (float32 and float64)."""
    g = _gen(seed + 7919)
    return _randn(g, case["m"], 3).float(), _randn(g, 12)


def _bandwidths(X, a_r):
    """sigma and softening a program starts its tuning from."""
    lam = float(torch.linalg.eigvalsh(torch.cov(X.double().T.cpu(), correction=0))[-1])
    return float(a_r.double().std(unbiased=False)), 0.05 * math.sqrt(lam)


def prepare(case, seed):
    ctx = _ctx()
    kind = case["kind"]
    st = {"ctx": ctx, "kind": kind, "case": case}
    if kind == "batch":
        pairs = _batch_pairs(case, seed)
        st["rf"] = [sg.Cloud(X) for X, _ in pairs]
        st["tm"] = [sg.Cloud(Y) for _, Y in pairs]
        st["prm"] = _params(case)
        return st
    X, Y, T = _pair(case, seed)
    if kind == "descriptors":
        st["rf"] = sg.Cloud(X)
        return st
    w, m = _masses(case, seed)
    st["rf"] = rf = sg.Cloud(X, w)
    st["tm"] = tm = sg.Cloud(Y, m)
    if kind in ("register", "multistart"):
        st["prm"] = _params(case)
        if kind == "multistart":
            st["R0"] = _rotations(case["S"])
        return st
    if kind in ("change", "residual"):
        st["pose"] = _inverse_pose(T, _gen(seed + 104729))
        if kind == "change":
            st["a_t"], st["a_r"] = ctx.descriptors(tm, case["k"])[0], ctx.descriptors(rf, case["k"])[0]
            st["sigma"] = float(st["a_r"].double().std(unbiased=False))
        return st
    if kind == "vector":
        st["mom_t"], st["mom_r"] = ctx.descriptors(tm, case["k"])[1], ctx.descriptors(rf, case["k"])[1]
        st["pose"] = sg.pose_identity()
        st["prm"] = sg.Params(p=1.0, k=case["k"], E=100)
        return st
    st["a_t"], st["mom_t"] = ctx.descriptors(tm, 16)
    st["a_r"], st["mom_r"] = ctx.descriptors(rf, 16)
    if kind == "step":
        st["pose"] = sg.pose_identity()
        st["prm"] = _params(case, k=16, E=100, eps=_soft(case, X))
        return st
    sigma, eps = _bandwidths(X, st["a_r"])
    st["sigma"], st["eps"] = sigma, eps
    if kind == "force_grad":
        gf, gw = _grads_in(case, seed)
        st["gf"], st["gw"] = gf, gw / case["m"]
        st["Y"] = Y.clone().requires_grad_(True)
        st["m"] = torch.ones(case["m"], device=DEV).requires_grad_(True)
        st["sig"] = torch.tensor(sigma, device=DEV, dtype=F64, requires_grad=True)
        st["ep"] = torch.tensor(eps, device=DEV, dtype=F64, requires_grad=True)
        st["prm"] = sg.Params(p=case["p"], k=16)
    else:
        st["gp"] = _grads_in(case, seed)[1].new_tensor(np.linspace(-1.0, 1.0, 13))
        st["sig"] = torch.tensor(sigma, dtype=F64, requires_grad=True)
        st["ep"] = torch.tensor(eps, dtype=F64, requires_grad=True)
        st["pose"] = sg.pose_identity().requires_grad_(True)
        st["prm"] = sg.Params(p=2.0, k=16, E=case["E"])
    return st


# -------------------------------------------------------------------- runs
def run(st):
    ctx, case, kind = st["ctx"], st["case"], st["kind"]
    if kind == "register":
        pose, _ = ctx.register(st["tm"], st["rf"], st["prm"])
        return {"pose": pose}
    if kind == "batch":
        poses, energy, _ = ctx.register_batch(st["tm"], st["rf"], st["prm"])
        return {"poses": poses, "energy": energy}
    if kind == "multistart":
        poses, energy, best = ctx.multistart(st["tm"], st["rf"], st["prm"], st["R0"])
        return {"poses": poses, "energy": energy, "best": best}
    if kind == "step":
        pose, wrench, f = ctx.step(st["tm"], st["a_t"], st["rf"], st["a_r"], st["mom_t"], st["mom_r"], st["prm"], 50,
                                   st["pose"], want_f=True)
        return {"pose": pose, "wrench": wrench, "f": f}
    if kind == "descriptors":
        a, mom = ctx.descriptors(st["rf"], case["k"])
        return {"a": a, "moments": mom}
    if kind == "vector":
        hX = ctx.descriptors_hn(st["rf"], case["k"], case["D"])
        hY = ctx.descriptors_hn(st["tm"], case["k"], case["D"])
        pose, _, f = ctx.step_vec(st["tm"], hY, st["rf"], hX, st["mom_t"], st["mom_r"], st["prm"], 50, st["pose"],
                                  want_f=True)
        return {"hX": hX, "hY": hY, "pose": pose, "f": f}
    if kind == "change":
        flags, nn, d2 = ctx.change_detect(st["tm"], st["a_t"], st["rf"], st["a_r"], st["pose"], case["tau"],
                                          st["sigma"], 0.5)
        return {"flags": flags, "nn": nn, "d2": d2}
    if kind == "residual":
        return {"rmse": ctx.residual(st["tm"], st["rf"], st["pose"])}
    if kind == "force_grad":
        f, w = sg.ForceField.apply(ctx, st["Y"], st["m"], st["sig"], st["ep"], st["a_t"], st["rf"], st["a_r"],
                                   st["mom_r"], st["prm"], 0.5 * G1)
        gy, gm, gs, ge = torch.autograd.grad([f, w], [st["Y"], st["m"], st["sig"], st["ep"]], [st["gf"], st["gw"]])
        return {"f": f.detach(), "wrench": w.detach(), "gy": gy, "gm": gm, "gsigma": gs, "geps": ge}
    pose = sg.UnrolledRegistration.apply(st["sig"], st["ep"], st["pose"], ctx, st["tm"], st["a_t"], st["rf"],
                                         st["a_r"], st["mom_t"], st["mom_r"], st["prm"], case["K"])
    gs, ge, gp = torch.autograd.grad(pose, [st["sig"], st["ep"], st["pose"]], st["gp"])
    return {"pose": pose.detach(), "gsigma": gs, "geps": ge, "gpose": gp}


def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the pair
    interactions the call is defined by (an FMA counts 2; 13 per pair for
    p = 1, 20 otherwise) or, where there is none, of its per-point part."""
    kind = case["kind"]
    pair = 13.0 if case.get("p", 1.0) == 1.0 else 20.0
    if kind == "batch":
        n = [int(round(math.exp(math.log(case["nmin"]) + (i + 0.5) / case["B"] *
                                math.log(case["nmax"] / case["nmin"])))) for i in range(case["B"])]
        return {"bytes": sum(12.0 * 2.1 * v for v in n) + 112.0 * case["B"], "flops": sum(pair * 1.1 * v * v for v in n)}
    n = float(case["n"])
    m = float(case.get("m", n))
    if kind == "descriptors":
        return {"bytes": 16.0 * n + 80, "flops": n * case["k"] * 30.0}
    if kind == "register":
        evals = 1 if case["flags"] & SUMS else case["E"]
        return {"bytes": 12.0 * (m + n) + 104, "flops": evals * pair * m * n}
    if kind == "multistart":
        return {"bytes": 12.0 * (m + n) + 72 * case["S"] + 116 * case["S"], "flops": pair * m * n}
    if kind == "step":
        return {"bytes": 16.0 * (m + n) + 12.0 * m + 208, "flops": pair * m * n}
    if kind == "vector":
        D = case["D"]
        return {"bytes": 12.0 * (m + n) + 4.0 * D * (m + n) + 12.0 * m, "flops": (2.0 * (D + 2) + 8.0) * m * n}
    if kind == "change":
        return {"bytes": 16.0 * (m + n) + 9.0 * m, "flops": 60.0 * m}
    if kind == "residual":
        return {"bytes": 12.0 * (m + n) + 8, "flops": 60.0 * m}
    if kind == "force_grad":
        return {"bytes": 16.0 * (m + n) + 12.0 * m + 28.0 * m, "flops": (pair + 30.0) * m * n}
    return {"bytes": 16.0 * (m + n), "flops": case["E"] * (2 * pair + 30.0) * m * n}


# ------------------------------------------------------- float64 evaluation
def _chunks(total, rows):
    rows = max(1, int(rows))
    return [(i, min(total, i + rows)) for i in range(0, total, rows)]


def _order(P):
    """Indices along a space-filling curve (neighbours in space stay near)."""
    lo, hi = P.amin(0), P.amax(0)
    q = ((P - lo) / (hi - lo).clamp(min=1e-30).amax() * 1023).long().clamp(0, 1023)
    code = torch.zeros(len(P), dtype=torch.int64, device=P.device)
    for b in range(10):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    return code.argsort()


def _keys(Q, X):
    """float32 squared distances ((dx*dx + dy*dy) + dz*dz), every operation rounded."""
    d = None
    for a in range(3):
        e = X[None, :, a] - Q[:, None, a]
        d = e * e if d is None else d + e * e
    return d


def _knn(P, k):
    """Neighbour lists (self included) by (float32 distance, index)."""
    n = len(P)
    out = torch.empty((n, k), dtype=torch.int64, device=P.device)
    order = _order(P)
    ids = torch.arange(n, device=P.device)
    ext = float((P.amax(0) - P.amin(0)).amax())
    for i, j in _chunks(n, 1024):
        q = order[i:j]
        Q = P[q]
        todo = torch.arange(len(q), device=P.device)
        lo, hi = Q.amin(0), Q.amax(0)
        r = max(1e-6, 2.0 * math.sqrt(k / n) * ext / 4)
        while len(todo):
            cand = ids[((P > lo - r) & (P < hi + r)).all(1)]
            if len(cand) >= k:
                rows = []
                for a, b in _chunks(len(todo), 6e7 // len(cand)):
                    d = _keys(Q[todo[a:b]], P[cand])
                    key = (d.view(torch.int32).long() << 32) | cand[None, :]
                    rows.append(torch.topk(key, k, dim=1, largest=False, sorted=True).values)
                best = torch.cat(rows)
                kth = (best[:, -1] >> 32).int().view(torch.float32)
                ok = (kth.double() * 1.0001 < r * r) | (len(cand) == n)
                out[q[todo[ok]]] = best[ok] & 0xFFFFFFFF
                todo = todo[~ok]
            r *= 2.0
    return out


def _covariances(P, nbr):
    Q = P.double()[nbr]
    Q = Q - Q.mean(1, keepdim=True)
    return Q.transpose(1, 2).contiguous() @ Q.contiguous() / nbr.shape[1]


def _curvature(P, k):
    """Smallest eigenvalue over the trace of every neighbourhood covariance
    (float64 values of the float32 results)."""
    C = _covariances(P, _knn(P, k))
    lam = torch.from_numpy(np.linalg.eigvalsh(C.cpu().numpy())).to(P.device)
    tr = lam.sum(1)
    return torch.where(tr > 0, lam[:, 0] / tr, torch.zeros_like(tr))


def _moments(P):
    Q = P.double()
    c = Q.mean(0)
    S = (Q - c).T @ (Q - c) / len(Q)
    lam = np.linalg.eigvalsh(S.cpu().numpy())[-1]
    return c, S, float(lam)


def _G(t, E):
    return 0.1 * G1 + 0.9 * G1 / (1.0 + math.exp(-((t - 1) - E / 2.0)))


class _Law:
    """Pair weights of eqs. 3, 10, 11 for one (reference, template) pair."""

    def __init__(self, X, aX, aY, p=1.0, g_mode=0, sigma=None, eps=0.0, w=None):
        self.X, self.aX, self.aY, self.p, self.eps = X.double(), aX, aY, p, eps
        self.shape = g_mode != 2
        flat = aX.dim() == 1
        abar = aX.mean(0)
        if sigma is None:
            sigma = aX.std(unbiased=False) if flat else ((aX - abar) ** 2).sum(1).mean().sqrt()
        self.sigma = sigma
        self.gX = aX / abar if g_mode == 1 else torch.ones(len(X), device=X.device, dtype=F64)
        self.gY = aY / abar if g_mode == 1 else torch.ones(len(aY), device=X.device, dtype=F64)
        if w is not None:
            self.gX = self.gX * w.double()
        self.c, _, self.lam = _moments(X)
        self.Z = len(X) if w is None else float(w.double().sum())
        self.rows = 4e7 // len(X)

    def similarity(self, i, j):
        if not self.shape:
            return self.gX.expand(j - i, -1)
        if self.aX.dim() == 1:
            d2 = (self.aY[i:j, None] - self.aX[None, :]) ** 2
        else:
            a, b = self.aY[i:j], self.aX
            d2 = sum((a[:, None, q] - b[None, :, q]) ** 2 for q in range(a.shape[1]))
        return torch.exp(-d2 / self.sigma ** 2) * self.gX[None, :]

    def sums(self):
        """sum_j c_ij (1, x_j, |x_j|^2) for p = 1, x relative to the centroid."""
        x = self.X - self.c
        V = torch.cat([torch.ones_like(x[:, :1]), x, (x * x).sum(1, keepdim=True)], 1)
        return torch.cat([self.similarity(i, j) @ V for i, j in _chunks(len(self.aY), self.rows)])

    def rows_force(self, Yc, i, j, x):
        """sum_j c_ij (y_i - x_j) h and the energy terms of rows i .. j."""
        s = self.similarity(i, j)
        r = [Yc[:, a, None] - x[None, :, a] for a in range(3)]
        q = r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + self.eps ** 2
        h = s if self.p == 1.0 else s * (q / self.lam) ** ((self.p - 1.0) / 2.0)
        f = torch.stack([(h * e).sum(1) for e in r], 1)
        return f * self.gY[i:j, None], (h * q).sum(1) * self.gY[i:j]

    def force(self, Y, G):
        """Per-point forces and the energy at template positions Y."""
        x = self.X - self.c
        out, U = [], 0.0
        for i, j in _chunks(len(Y), self.rows / 4):
            f, u = self.rows_force((Y - self.c)[i:j], i, j, x)
            out.append(f)
            U = U + u.sum()
        return -(G / self.Z) * torch.cat(out), G / self.Z / (self.p + 1.0) * U


def _update(pose, Ybar, F, K, M, S0, lamX, lamY0, dt2, mass=None):
    """One rigid update (eqs. 5.5, 6, 8, 9, and one Newton-Schulz step back
    to a rotation) of the pose [13] (torch float64, CPU)."""
    s, R, t = pose[0], pose[1:10].view(3, 3), pose[10:]
    yb = s * R @ Ybar + t
    C = M * s * s * R @ S0 @ R.T + dt2 * K
    U, _, Vh = torch.linalg.svd(C)
    sign = torch.sign(torch.linalg.det(Vh.T @ U.T)).detach()
    Rk = Vh.T @ torch.diag(torch.stack([torch.ones_like(sign), torch.ones_like(sign), sign])) @ U.T
    c = math.sqrt(lamX / lamY0) / s
    Rn = Rk.T @ R
    Rn = 0.5 * Rn @ (3.0 * torch.eye(3, dtype=F64) - Rn.T @ Rn)
    return torch.cat([(c * s).reshape(1), Rn.reshape(-1), c * Rk.T @ (t - yb) + yb + dt2 * F / (mass or M)])


def _iterate_sums(Y0, law, S, E, pose):
    """E iterations of the p = 1 law from its pair sums; (pose, last energy)."""
    Y0 = Y0.double()
    M = len(Y0)
    c0, S0, lamY0 = _moments(Y0)
    e = Y0 - c0
    g = law.gY[:, None]
    c0c, S0c, U = c0.cpu(), S0.cpu(), None
    for t in range(E):
        G = _G(t, E)
        P = pose.to(Y0.device)
        A = P[0] * P[1:10].view(3, 3)
        y = e @ A.T
        yc = y + (A @ c0 + P[10:] - law.c)
        f = -(G / law.Z) * g * (yc * S[:, :1] - S[:, 1:4])
        if t == E - 1:
            U = G / law.Z / 2.0 * (law.gY * (((yc * yc).sum(1) + law.eps ** 2) * S[:, 0] -
                                             2 * (yc * S[:, 1:4]).sum(1) + S[:, 4])).sum()
        W = torch.cat([f.sum(0), (f.T @ y).reshape(-1)]).cpu()
        pose = _update(pose, c0c, W[:3], W[3:].view(3, 3), M, S0c, law.lam, lamY0, 1.0 / G1)
    return pose, U


def _identity():
    return torch.tensor([1.0, 1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], dtype=F64)


def _register_exact(X, Y, k, g_mode, E, poses=None):
    law = _Law(X, _curvature(X, k).float().double(), _curvature(Y, k).float().double(), g_mode=g_mode)
    S = law.sums()
    if poses is None:
        return _iterate_sums(Y, law, S, E, _identity())
    return [_iterate_sums(Y, law, S, E, p) for p in poses]


def _step_exact(Y, law, t, E, m=None):
    c0, S0, lamY0 = _moments(Y)
    f, U = law.force(Y.double(), _G(t, E))
    e = Y.double() - c0
    F = f.sum(0) if m is None else (m.double()[:, None] * f).sum(0)
    W = torch.cat([F, (f.T @ e).reshape(-1), U.reshape(1)])
    Wc = W.cpu()
    pose = _update(_identity(), c0.cpu(), Wc[:3], Wc[3:12].view(3, 3), len(Y), S0.cpu(), law.lam, lamY0, 1.0 / G1,
                   None if m is None else float(m.double().sum()))
    return pose, W, f


def _histograms(P, k, D):
    nbr = _knn(P, k)
    nv = torch.from_numpy(np.linalg.eigh(_covariances(P, nbr).cpu().numpy())[1][:, :, 0].copy()).to(P.device)
    u = (nv[nbr] * nv[:, None, :]).sum(2).abs().clamp(max=1.0)
    c = torch.arange(D, device=P.device, dtype=F64) / (D - 1)
    return (1.0 - (D - 1) * (u[:, :, None] - c).abs()).clamp(min=0.0).mean(1)


def _nearest(Q, X):
    """Nearest reference point of float32 points Q by the float32 key."""
    idx = []
    for i, j in _chunks(len(Q), 2e8 // len(X)):
        idx.append(_keys(Q[i:j], X).argmin(1))
    return torch.cat(idx)


def _posed(Y, pose):
    return pose[0] * Y.double() @ pose[1:10].view(3, 3).T + pose[10:]


def _field_vjp(law_of, Y, lam, G, sigma, eps):
    """sum_i lam_i . f_i(y_i; sigma, eps): gradients by autograd, row block by row block."""
    sg_, ep_ = (torch.tensor(float(v), device=DEV, dtype=F64, requires_grad=True) for v in (sigma, eps))
    gY, gs, ge = torch.empty_like(Y), 0.0, 0.0
    law = law_of(sg_, ep_)
    x = law.X - law.c
    for i, j in _chunks(len(Y), law.rows / 8):
        y = Y[i:j].clone().requires_grad_(True)
        f, _ = law.rows_force(y - law.c, i, j, x)
        loss = -(G / law.Z) * (lam[i:j] * f).sum()
        a, b, c = torch.autograd.grad(loss, [y, sg_, ep_], allow_unused=True)
        gY[i:j] = a
        gs = gs + b
        ge = ge + (c if c is not None else 0.0)
    return gY, gs, torch.as_tensor(ge, device=DEV, dtype=F64)


def _force_grad_exact(case, seed):
    X, Y, _ = _pair(case, seed)
    aX, aY = (_curvature(P, 16).float().double() for P in (X, Y))
    sigma, eps = _bandwidths(X, aX)
    G, m = 0.5 * G1, case["m"]
    law_of = lambda s, e: _Law(X, aX, aY, case["p"], 0, s, e)  # noqa: E731
    Y = Y.double()
    f, _ = law_of(torch.tensor(sigma, device=DEV, dtype=F64), eps).force(Y, G)
    gf, gw = _grads_in(case, seed)
    gf, gw = gf.double(), gw / m
    gF, gK = gw[:3], gw[3:].view(3, 3)
    e = Y - Y.mean(0)
    gY, gs, ge = _field_vjp(law_of, Y, gf + gF + e @ gK.T, G, sigma, eps)
    gY = gY + (f - f.mean(0)) @ gK
    return {"f": f, "wrench": torch.cat([f.sum(0), (f.T @ e).reshape(-1)]), "gy": gY, "gm": f @ gF, "gsigma": gs,
            "geps": ge}


def _unrolled_exact(case, seed):
    X, Y, _ = _pair(case, seed)
    aX, aY = (_curvature(P, 16).float().double() for P in (X, Y))
    sigma, eps = _bandwidths(X, aX)
    E, M = case["E"], case["m"]
    law_of = lambda s, e: _Law(X, aX, aY, 2.0, 0, s, e)  # noqa: E731
    law = law_of(torch.tensor(sigma, device=DEV, dtype=F64), eps)
    Y0 = Y.double()
    c0, S0, lamY0 = _moments(Y0)
    c0c, S0c = c0.cpu(), S0.cpu()
    poses, wrench = [_identity()], []
    for t in range(E):
        y = _posed(Y0, poses[-1].to(DEV))
        f, _ = law.force(y, _G(t, E))
        wrench.append(torch.cat([f.sum(0), (f.T @ (y - y.mean(0))).reshape(-1)]).cpu())
        W = wrench[-1]
        poses.append(_update(poses[-1], c0c, W[:3], W[3:].view(3, 3), M, S0c, law.lam, lamY0, 1.0 / G1))
    g = torch.linspace(-1.0, 1.0, 13, dtype=F64)
    gs, ge = 0.0, 0.0
    for t in reversed(range(E)):
        p = poses[t].clone().requires_grad_(True)
        W = wrench[t].clone().requires_grad_(True)
        q = _update(p, c0c, W[:3], W[3:].view(3, 3), M, S0c, law.lam, lamY0, 1.0 / G1)
        gp, gW = torch.autograd.grad(q, [p, W], g)
        gW = gW.to(DEV)
        y = _posed(Y0, poses[t].to(DEV))
        yc = y - y.mean(0)
        lam = gW[:3] + yc @ gW[3:].view(3, 3).T
        gy, a, b = _field_vjp(law_of, y, lam, _G(t, E), sigma, eps)
        f, _ = law.force(y, _G(t, E))
        gy = gy + (f - f.mean(0)) @ gW[3:].view(3, 3)
        p = poses[t].to(DEV).requires_grad_(True)
        back = torch.autograd.grad((_posed(Y0, p) * gy).sum(), p)[0]
        g = gp + back.cpu()
        gs, ge = gs + a, ge + b
    return {"pose": poses[-1], "gsigma": gs, "geps": ge, "gpose": g}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if case["B"] * case["nmax"] ** 2 > 3e11:
            return None
        got = [_register_exact(X, Y, case["k"], 0, case["E"]) for X, Y in _batch_pairs(case, seed)]
        return {"poses": torch.stack([p for p, _ in got]), "energy": torch.stack([u.cpu() for _, u in got])}
    if kind == "force_grad":
        return _force_grad_exact(case, seed)
    if kind == "unrolled":
        return _unrolled_exact(case, seed)
    X, Y, T = _pair(case, seed)
    if kind == "register":
        return {"pose": _register_exact(X, Y, case["k"], case["g_mode"], case["E"])[0]}
    if kind == "multistart":
        c0 = _moments(Y)[0].cpu()
        starts = []
        for R in torch.as_tensor(_rotations(case["S"])):
            starts.append(torch.cat([torch.ones(1, dtype=F64), R.reshape(-1), c0 - R @ c0]))
        got = _register_exact(X, Y, case["k"], 0, case["E"], starts)
        return {"poses": torch.stack([p for p, _ in got]), "energy": torch.stack([u.cpu() for _, u in got]),
                "best": None}
    if kind == "descriptors":
        c, S, lam = _moments(X)
        six = torch.stack([S[0, 0], S[1, 1], S[2, 2], S[0, 1], S[0, 2], S[1, 2], S.new_tensor(lam)])
        return {"a": _curvature(X, case["k"]), "moments": torch.cat([c, six])}
    if kind == "step":
        w, m = _masses(case, seed)
        law = _Law(X, *(_curvature(P, 16).float().double() for P in (X, Y)), case["p"], case["g_mode"], None,
                   _soft(case, X), w)
        pose, W, f = _step_exact(Y, law, 50, 100, m)
        if case["flags"] & 2:
            W[12] = 0.0  # mixed precision reports no energy
        return {"pose": pose, "wrench": W, "f": f}
    if kind == "vector":
        hX, hY = (_histograms(P, case["k"], case["D"]) for P in (X, Y))
        law = _Law(X, hX.float().double(), hY.float().double())
        pose, _, f = _step_exact(Y, law, 50, 100)
        return {"hX": hX, "hY": hY, "pose": pose, "f": f}
    pose = _inverse_pose(T, _gen(seed + 104729))
    y = _posed(Y, pose)
    nn = _nearest(y.float(), X)
    d = (y - X.double()[nn]).square().sum(1)
    if kind == "residual":
        return {"rmse": d.mean().sqrt().reshape(1)}
    d = (y.float().double() - X.double()[nn]).square().sum(1)
    d = torch.where(d.float() <= np.float32(case["tau"] ** 2), d, torch.full_like(d, math.inf))
    return {"flags": None, "nn": None, "d2": d}
