"""Performance cases of the simulator: what a user's program runs, through the public
entry points, over the range of sizes this repository's workloads and tests cover.

Each case is a dict of plain values.  ``prepare`` makes what such a program holds before
the call (model, parameters, start state, target); ``run`` is one call of it; ``work``
counts the bytes of its inputs and outputs and the operations of its steps; ``exact``
evaluates the same inputs in float64 with plain torch operations written here.

Meshes belong to the case (``mesh_seed``); materials, masses, start states, targets,
controller weights and image gradients are drawn from the seed given to ``prepare``.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2104_02646_amd import autograd, gsim, serve
from paper_2104_02646_amd import workloads as W

EXEC = {"plain": gsim.EXEC_PLAIN, "graph": gsim.EXEC_GRAPH, "persist": gsim.EXEC_PERSIST}
OMEGA, ACT_SCALE, SIGNALS = 2 * math.pi * 4.0, 0.05, 8  # controller of the control tasks
# arithmetic of one element (or particle) in one step, forward and adjoint
FLOPS = {"tet": (230, 620), "tri": (130, 350), "hinge": (220, 600), "particle": (40, 90)}


def listed():
    return [
        # one simulation step of one small body: the smallest call, an interactive loop
        {"name": "cube step", "kind": "step", "mesh": "cube", "steps": 1},
        # the README's program: one small body's gradient through autograd, default settings
        {"name": "cube gradient", "kind": "gradient", "mesh": "cube", "steps": 100, "every": 10, "exec": "plain",
         "via": "autograd"},
        # control tasks (up to the first contacts: beyond them the loss is not locally linear):
        # controller -> actuated rollout -> loss -> adjoint -> weight gradient;
        # the walker (168 tets) in the execution the tuner takes for a body of one tile
        {"name": "walker control", "kind": "control", "mesh": "walker", "steps": 60, "every": 20, "exec": "persist"},
        # the soft gear (1152 tets) on the graph path
        {"name": "gear control", "kind": "control", "mesh": "gear", "steps": 60, "every": 20, "exec": "graph"},
        # one cloth with bending: membrane stiffness and mass estimation
        {"name": "cloth gradient", "kind": "gradient", "mesh": "cloth", "side": 64, "steps": 100, "every": 10,
         "exec": "graph", "via": "model"},
        # a batch of free cloths under lift/drag: initial-velocity gradients
        {"name": "thrown cloths", "kind": "gradient", "mesh": "air", "bodies": 16, "mesh_seed": 900, "steps": 100,
         "every": 10, "exec": "plain", "via": "model"},
        # one large body
        {"name": "blob gradient", "kind": "gradient", "mesh": "blob", "tets": 200000, "steps": 100, "every": 25,
         "exec": "graph", "via": "model"},
        # forward prediction only, a ragged batch in the library's default tiles and lanes
        {"name": "batch rollout", "kind": "rollout", "mesh": "batch", "bodies": 64, "lo": 500, "hi": 20000,
         "mesh_seed": 21, "steps": 100, "every": 10, "exec": "graph"},
        # parameter estimation over a batch, as the benchmark's workload in its tuned settings
        {"name": "batch gradient", "kind": "gradient", "mesh": "batch", "bodies": 256, "lo": 500, "hi": 20000,
         "mesh_seed": 20, "steps": 100, "every": 10, "exec": "graph", "via": "model", "tile": 512, "lanes": 4},
        # rigid parameter estimation, in the precision that gradients through bouncing need
        {"name": "rigid batch", "kind": "rigid", "bodies": 1024, "mesh_seed": 80, "steps": 150, "dtype": "f64"},
        # pixel loss: soft silhouette of the cloth and its adjoint
        {"name": "silhouette", "kind": "silhouette", "side": 64, "height": 256, "width": 256, "sigma": 1.0},
        # continuous batching: a burst of tet and cloth gradient queries
        {"name": "query burst", "kind": "serve", "queries": 12, "mesh_seed": 40, "max_steps": 120, "every": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "gradient", "gradient", "batch", "rollout", "control", "air", "rigid", "silhouette",
                       "serve"])
    if kind == "step":
        return {"kind": "step", "mesh": "batch", "bodies": rng.randint(1, 3), "lo": 100, "hi": _log(rng, 300, 20000),
                "mesh_seed": rng.randint(1, 999), "steps": _log(rng, 1, 20)}
    if kind == "gradient":
        c = {"kind": "gradient", "steps": _log(rng, 10, 150), "every": rng.randint(1, 25),
             "exec": rng.choice(["plain", "graph"]), "via": rng.choice(["model", "autograd"])}
        if rng.random() < 0.4:
            return dict(c, mesh="cloth", side=rng.randint(5, 96), mesh_seed=rng.randint(1, 999))
        return dict(c, mesh="batch", bodies=1, lo=60, hi=_log(rng, 100, 60000), mesh_seed=rng.randint(1, 999))
    if kind in ("batch", "rollout"):
        c = {"kind": "rollout" if kind == "rollout" else "gradient", "mesh": "batch", "bodies": _log(rng, 2, 96),
             "lo": _log(rng, 100, 1000), "hi": _log(rng, 2000, 20000), "mesh_seed": rng.randint(1, 999),
             "steps": rng.randint(20, 100), "every": rng.randint(3, 20), "exec": "graph",
             "tile": rng.choice([128, 256, 384, 512]), "lanes": rng.randint(1, 2)}
        return dict(c, via="model") if kind == "batch" else c
    if kind == "control":
        return {"kind": "control", "mesh": rng.choice(["walker", "gear"]), "steps": _log(rng, 10, 60),
                "every": rng.randint(5, 30), "exec": rng.choice(["plain", "graph", "persist"])}
    if kind == "air":
        return {"kind": "gradient", "mesh": "air", "bodies": _log(rng, 1, 24), "mesh_seed": rng.randint(1, 999),
                "steps": _log(rng, 10, 100), "every": rng.randint(4, 20), "exec": rng.choice(["plain", "graph"]),
                "via": "model"}
    if kind == "rigid":
        f64 = rng.random() < 0.5
        return {"kind": "rigid", "bodies": _log(rng, 1, 1024), "mesh_seed": rng.randint(1, 999),
                "steps": _log(rng, 10, 150 if f64 else 60), "dtype": "f64" if f64 else "f32"}
    if kind == "silhouette":
        return {"kind": "silhouette", "side": rng.randint(8, 128), "height": _log(rng, 60, 700),
                "width": _log(rng, 60, 700), "sigma": rng.uniform(0.5, 2.0)}
    return {"kind": "serve", "queries": rng.randint(1, 12), "mesh_seed": rng.randint(1, 999),
            "max_steps": rng.randint(60, 120), "every": rng.randint(5, 20)}


# ------------------------------------------------------------------ inputs ---
@functools.lru_cache(maxsize=8)
def _meshes(key):
    c = dict(key)
    seed = c.get("mesh_seed", 0)
    if c["mesh"] == "cube":
        return [W.tiny_cube(0)]
    if c["mesh"] == "walker":
        return [W.walker()]
    if c["mesh"] == "gear":
        return [W.gear()]
    if c["mesh"] == "cloth":
        return [W.cloth(10, n=c["side"])]
    if c["mesh"] == "blob":
        return [W.large_blob(30, c["tets"])]
    if c["mesh"] == "air":
        return [W.control_cloth(1000 * seed + i) for i in range(c["bodies"])]
    return [W.batch_body(1000 * seed + i, lo=c["lo"], hi=c["hi"]) for i in range(c["bodies"])]


def _redraw(b, rng, spread):
    """The mesh of b with materials, masses and start velocities of this seed, rounded to
    float32 so that the float64 evaluation sees the same inputs."""
    kw = {"v0": b.v0 + rng.normal(0.0, 0.05, 3) + rng.normal(0.0, 1e-3, b.v0.shape)}
    if b.ne:
        lo, hi = spread
        kw["mu"], kw["lam"] = (np.exp(rng.uniform(np.log(lo), np.log(hi), b.ne)) for _ in range(2))
    if b.nt:
        kw["ktri"] = rng.uniform(1e3, 1e4, b.nt)
    kw["mass"] = b.mass * rng.uniform(0.9, 1.1, b.np)
    return b.with_params(**kw).round_to(np.float32)


def _bodies(case, seed):
    rng = np.random.default_rng(seed)
    key = tuple(sorted((k, case[k]) for k in ("mesh", "mesh_seed", "bodies", "lo", "hi", "side", "tets") if k in case))
    spread = {"blob": (1e4, 1e6), "gear": (5e4, 1.5e5), "walker": (5e4, 1.5e5)}.get(case["mesh"], (1e4, 1e5))
    out = []
    for b in _meshes(key):
        b = _redraw(b, rng, spread)
        t = b.x0 + np.array([0.0, -0.05, 0.0]) + rng.normal(0.0, 0.005, b.x0.shape)
        out.append(b.with_params(target=t.astype(np.float32).astype(np.float64)))
    return out


def _weights(case, bodies, seed):
    w = W.controller_weights(seed + 1, SIGNALS, sum(b.ne for b in bodies))
    return w.astype(np.float32)


def _rigid_bodies(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(case["bodies"]):
        b = W.rigid_body(100000 * case["mesh_seed"] + i)
        s = b.s0.copy()
        s[1] -= 0.15
        s[7:13] += rng.normal(0.0, 0.2, 6)
        b.s0, b.mass = s, b.mass * rng.uniform(0.9, 1.1)
        b.inertia = b.inertia * rng.uniform(0.9, 1.1)
        out.append(b.round_to(np.float32))
    t = np.concatenate([b.verts + b.s0[:3] + rng.normal(0.0, 0.1, 3) for b in out])
    return out, t.astype(np.float32).astype(np.float64)


def _view(case, seed):
    """The cloth's mesh, its bent positions [3, n], the camera matrix and the image gradient."""
    rng = np.random.default_rng(seed)
    b = W.cloth(10, n=case["side"])
    x = b.X + np.stack([np.zeros(b.np), 0.15 * np.sin(3 * b.X[:, 0] + rng.uniform(0, 6)), np.zeros(b.np)], 1)
    x = (x + rng.normal(0.0, 0.15 / case["side"], x.shape)).astype(np.float32)
    h, w = case["height"], case["width"]
    eye, at = np.array([1.0, 3.0, 4.0]), np.array([1.0, 0.6, 1.0])
    f = (at - eye) / np.linalg.norm(at - eye)
    r = np.cross(f, [0.0, 1.0, 0.0])
    r /= np.linalg.norm(r)
    R = np.stack([r, np.cross(f, r), f])
    k = 1.1 * min(h, w)
    P = np.array([[k, 0, w / 2], [0, k, h / 2], [0, 0, 1.0]]) @ np.concatenate([R, (-R @ eye)[:, None]], 1)
    P = P.astype(np.float32).astype(np.float64)
    ibar = rng.uniform(-1.0, 1.0, (h, w)).astype(np.float32)
    return b.tris, np.ascontiguousarray(x.T), P, float(np.float32(case["sigma"])), ibar


def _queries(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for q in W.serving_trace(case["mesh_seed"], case["queries"]):
        if q.kind == "tet":
            b = W.batch_body(q.seed, lo=min(q.size, 20000), hi=min(q.size, 20000))
        else:
            b = W.cloth(10, n=min(q.size, 96))
        b = _redraw(b, rng, (1e4, 1e5))
        t = b.x0 + np.array([0.0, -0.05, 0.0]) + rng.normal(0.0, 0.005, b.x0.shape)
        out.append((b.with_params(target=t.astype(np.float32).astype(np.float64)), min(q.steps, case["max_steps"])))
    return out


def _cat(bodies, name, dtype=torch.float32):
    return gsim.soa(np.concatenate([getattr(b, name) for b in bodies]), dtype)


@functools.lru_cache(maxsize=1)
def _stream():
    """The program's own stream (graph execution needs one that is not the default)."""
    return torch.cuda.Stream()


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "steps": case.get("steps", 0)}
    if kind == "serve":
        s["engine"] = serve.Engine(pool_bytes=2 << 30, max_live=64)
        s["queries"] = [serve.QueryBuffers(b, t, case["every"]) for b, t in _queries(case, seed)]
        return s
    if kind == "silhouette":
        tris, x, s["P"], s["sigma"], ibar = _view(case, seed)
        s["x"] = torch.as_tensor(x, device="cuda")
        s["ibar"] = torch.as_tensor(ibar, device="cuda")
        s["renderer"] = gsim.Renderer(tris, x.shape[1], case["height"], case["width"])
        return s
    if kind == "rigid":
        bodies, target = _rigid_bodies(case, seed)
        dt = torch.float64 if case["dtype"] == "f64" else torch.float32
        s["model"] = m = gsim.RigidModel(bodies, dt)
        s["p"], s["s0"] = m.params_from_bodies(), m.initial_state()
        s["target"] = torch.as_tensor(target, dtype=dt, device="cuda")
        s["traj"], s["g"] = m.new_trajectory(case["steps"]), m.zero_grads()
        return s
    bodies = _bodies(case, seed)
    s["stream"] = _stream()
    s["via"] = case.get("via", "model")
    with torch.cuda.stream(s["stream"]):
        T = case["steps"]
        s["model"] = m = gsim.Model(bodies, torch.float32, max_steps=T, ckpt_every=case.get("every", T),
                                    tile_elems=case.get("tile", 0))
        m.set_exec(EXEC[case.get("exec", "plain")])
        if "lanes" in case:
            m.set_lanes(case["lanes"])
        s["p"] = m.params_from_bodies()
        s["x0"], s["v0"], s["target"] = (_cat(bodies, k) for k in ("x0", "v0", "target"))
        if s["via"] == "autograd":
            s["wrt"] = [s["p"][k].requires_grad_(True) for k in sorted(s["p"])] + [s["x0"].requires_grad_(True),
                                                                                   s["v0"].requires_grad_(True)]
        else:
            s["out"], s["adj"] = m.empty_state(), m.empty_state()
            s["g"] = m.zero_grads()
        if kind == "control":
            s["W"] = torch.as_tensor(_weights(case, bodies, seed), device="cuda")
            s["dt"] = bodies[0].dt
            s["act"], s["gact"] = (torch.zeros(T, m.ne, device="cuda") for _ in range(2))
            s["gW"] = torch.zeros_like(s["W"])
    s["stream"].synchronize()
    return s


# ------------------------------------------------------------------ a pass ---
def run(s):
    kind = s["kind"]
    if kind == "serve":
        for q in s["queries"]:
            s["engine"].submit(q)
        s["engine"].run_until_idle()
        return [{"loss": q.loss, **{k: v for k, v in q.out.items() if v.size}} for q in s["queries"]]
    if kind == "silhouette":
        x = s["x"].detach().requires_grad_(True)
        image = autograd.render(s["renderer"], x, s["P"], s["sigma"])
        return {"image": image.detach(), "x": torch.autograd.grad(image, x, s["ibar"])[0]}
    if kind == "rigid":
        m, g = s["model"], s["g"]
        m.rollout(s["p"], s["s0"], s["steps"], traj=s["traj"])
        loss, sbar = m.loss(s["traj"][-1], s["target"])
        for t in g.values():
            t.zero_()
        return {"final": s["traj"][-1], "loss": loss, "s0": m.rollout_backward(s["p"], s["traj"], s["steps"], sbar, g),
                **g}
    m, T = s["model"], s["steps"]
    with torch.cuda.stream(s["stream"]):
        if kind == "step":
            return m.step(s["p"], s["x0"], s["v0"], T, out=s["out"])
        if kind == "rollout":
            return m.rollout(s["p"], s["x0"], s["v0"], T, checkpoint=False, out=s["out"])
        if s["via"] == "autograd":
            xT, vT = autograd.rollout(m, s["p"], s["x0"], s["v0"], T)
            loss = ((xT - s["target"]) ** 2).sum() / m.np
            return [loss.detach(), xT.detach(), vT.detach(), *torch.autograd.grad(loss, s["wrt"])]
        p, g = s["p"], s["g"]
        if kind == "control":
            gsim.controller_forward(s["W"], OMEGA, s["dt"], T, scale=ACT_SCALE, out=s["act"])
            s["gact"].zero_()
            p, g = dict(p, act=s["act"]), dict(g, act=s["gact"])
        x, v = m.rollout(p, s["x0"], s["v0"], T, out=s["out"])
        loss, xb, vb = m.loss_mse(x, s["target"])
        for t in s["g"].values():
            t.zero_()
        x0b, v0b = m.rollout_backward(p, T, xb, vb, g, out=s["adj"])
        out = {"loss": loss, "x": x, "v": v, "x0": x0b, "v0": v0b, **s["g"]}
        if kind == "control":
            s["gW"].zero_()
            out["W"] = gsim.controller_backward(s["W"], s["gact"], OMEGA, s["dt"], scale=ACT_SCALE, W_grad=s["gW"])
    return out


# -------------------------------------------------------------------- work ---
def _fem_work(bodies, T, gradient):
    ne, nt, nh, n = (sum(getattr(b, k) for b in bodies) for k in ("ne", "nt", "nh", "np"))
    counts = {"tet": ne, "tri": nt, "hinge": nh, "particle": n}
    flops = T * sum(c * (FLOPS[k][0] + (FLOPS[k][1] if gradient else 0)) for k, c in counts.items())
    # element records (corner indices, rest shape) and parameters, states in and out, mass
    nbytes = 4 * (16 * ne + 9 * nt + 5 * nh + 13 * n)
    if gradient:  # parameter gradients, target, state adjoints
        nbytes += 4 * (2 * ne + nt + n + 3 * n + 6 * n)
    return {"bytes": nbytes, "flops": flops}


def work(case):
    kind = case["kind"]
    if kind == "serve":
        ws = [_fem_work([b], t, True) for b, t in _queries(case, 0)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "silhouette":
        n, tris = case["side"] ** 2, 2 * (case["side"] - 1) ** 2
        px = case["height"] * case["width"]
        # ~60 operations where a triangle reaches a pixel, forward and adjoint; its reach is
        # its own area and the cut-off band around it
        side = 0.55 * min(case["height"], case["width"]) / case["side"]
        reach = (side + 2 * math.sqrt(13.8 * case["sigma"])) ** 2
        return {"bytes": 4 * (6 * n + 3 * tris + 2 * px), "flops": 130 * tris * reach}
    if kind == "rigid":
        bodies = [W.rigid_body(100000 * case["mesh_seed"] + i) for i in range(case["bodies"])]
        nv, nb, T = sum(b.nv for b in bodies), len(bodies), case["steps"]
        e = 8 if case["dtype"] == "f64" else 4
        return {"bytes": e * (6 * nv + nb * (13 * (T + 1) + 13 + 22 + 13)), "flops": T * (250 * nv + 1500 * nb)}
    bodies = _bodies(case, 0)
    w = _fem_work(bodies, case["steps"], kind in ("gradient", "control"))
    if kind == "control":
        n = sum(b.ne for b in bodies)
        w["bytes"] += 4 * 2 * SIGNALS * n
        w["flops"] += case["steps"] * n * 60
    return w


# ------------------------------------------------------------------- exact ---
def _dot(a, b):
    return (a * b).sum(-1)


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dtype)


class _Reference:
    """The step of the model's description (include/gsim.h) on a batch of bodies, float64."""

    def __init__(self, bodies):
        off = np.cumsum([0] + [b.np for b in bodies])
        cat = lambda a: np.concatenate(list(a))  # noqa: E731
        self.X, self.n = _t(cat(b.X for b in bodies)), int(off[-1])
        self.tets, self.tris, self.hinges = (_t(cat(getattr(b, k) + o for b, o in zip(bodies, off)), torch.int64)
                                             for k in ("tets", "tris", "hinges"))
        self.body = _t(np.repeat(np.arange(len(bodies)), np.diff(off)), torch.int64)
        self.free = (_t(cat(b.pinned for b in bodies))[:, None] == 0).double()
        self.dt, self.g, self.plane = (_t([getattr(b, k) for b in bodies])[self.body] for k in ("dt", "gravity", "plane"))
        self.dt = self.dt[:, None]
        self.on = _t([b.ground for b in bodies], torch.bool)[self.body, None]
        self.kb = _t([b.kb for b in bodies])
        self.contact_bodies, self.air = any(b.ground for b in bodies), any(b.air for b in bodies)
        if len(self.tets):
            X = self.X[self.tets]
            D = [X[:, i] - X[:, 0] for i in (1, 2, 3)]  # columns of Dm; rows of its inverse:
            det = _dot(D[0], _cross(D[1], D[2]))
            self.Di = [_cross(D[(i + 1) % 3], D[(i + 2) % 3]) / det[:, None] for i in range(3)]
            self.V = det.abs() / 6
        if len(self.tris):
            X = self.X[self.tris]
            d0, d1 = X[:, 1] - X[:, 0], X[:, 2] - X[:, 0]
            e0 = d0 / _dot(d0, d0).sqrt()[:, None]
            a, b = _dot(d0, e0), _dot(d1, e0)
            h = _dot(d1 - e0 * b[:, None], d1 - e0 * b[:, None]).sqrt()
            self.Ti, self.area = (1 / a, -b / (a * h), 1 / h), a * h / 2
        if len(self.hinges):
            self.phi0 = self._hinge(self.X[self.hinges])[0]
            self.hkb = self.kb[self.body[self.hinges[:, 0]]]

    @staticmethod
    def _hinge(x):
        x0, x1, x2, x3 = x.unbind(1)
        E, N1, N2 = x3 - x2, _cross(x0 - x2, x0 - x3), _cross(x1 - x3, x1 - x2)
        el, q1, q2 = _dot(E, E).sqrt(), _dot(N1, N1), _dot(N2, N2)
        Eh, a1, a2 = E / el[:, None], N1 / q1[:, None], N2 / q2[:, None]
        s = [_dot(x0 - x3, Eh), _dot(x1 - x3, Eh), _dot(x0 - x2, Eh), _dot(x1 - x2, Eh)]
        u = [a1 * el[:, None], a2 * el[:, None], a1 * s[0][:, None] + a2 * s[1][:, None],
             -(a1 * s[2][:, None] + a2 * s[3][:, None])]
        phi = torch.atan2(-_dot(_cross(N1, N2), Eh), _dot(N1, N2))
        return phi, el * el / (q1.sqrt() + q2.sqrt()), torch.stack(u, 1)

    def step(self, x, v, p, act):
        f = torch.zeros_like(x)
        if len(self.tets):
            c = x[self.tets]
            d = [c[:, i] - c[:, 0] for i in (1, 2, 3)]
            F = [d[0] * self.Di[0][:, j, None] + d[1] * self.Di[1][:, j, None] + d[2] * self.Di[2][:, j, None]
                 for j in range(3)]
            C = [_cross(F[1], F[2]), _cross(F[2], F[0]), _cross(F[0], F[1])]
            Ic, J = sum(_dot(a, a) for a in F), _dot(F[0], C[0])
            alpha = 1 + 0.75 * p["mu"] / p["lam"] + (act if act is not None else 0)
            A, B = (p["mu"] * (1 - 1 / (Ic + 1)))[:, None], (p["lam"] * (J - alpha))[:, None]
            Pk = [A * F[j] + B * C[j] for j in range(3)]
            fi = [-self.V[:, None] * sum(Pk[j] * self.Di[i][:, j, None] for j in range(3)) for i in range(3)]
            fe = torch.stack([-(fi[0] + fi[1] + fi[2]), *fi], 1)
            f = f.index_add(0, self.tets.reshape(-1), fe.reshape(-1, 3))
        if len(self.tris):
            c = x[self.tris]
            d0, d1 = c[:, 1] - c[:, 0], c[:, 2] - c[:, 0]
            i00, i01, i11 = (a[:, None] for a in self.Ti)  # Dm^-1 = [[i00, i01], [0, i11]]
            F0, F1 = d0 * i00, d0 * i01 + d1 * i11
            N = _cross(F0, F1)
            J = _dot(N, N).sqrt()[:, None]
            n = N / J
            A = p["ktri"][:, None] * (1 - 1 / (_dot(F0, F0) + _dot(F1, F1) + 1))[:, None]
            B = p["ktri"][:, None] * (J - 5 / 3)
            P0, P1 = A * F0 + B * _cross(F1, n), A * F1 + B * _cross(n, F0)
            f1, f2 = -self.area[:, None] * (P0 * i00 + P1 * i01), -self.area[:, None] * P1 * i11
            fe = torch.stack([-(f1 + f2), f1, f2], 1)
            if self.air:
                Nx = _cross(d0, d1)
                nn = _dot(Nx, Nx).sqrt()[:, None]
                n, A, u = Nx / nn, nn / 2, v[self.tris].mean(1)
                k = p["air"][self.body[self.tris[:, 0]]]
                sn, q = _dot(n, u)[:, None], _dot(u, u)[:, None]
                Fa = -A * (k[:, :1] * sn.abs() * u + k[:, 1:] * sn * (q * n - sn * u) / q.sqrt())
                fe = fe + Fa[:, None] / 3
            f = f.index_add(0, self.tris.reshape(-1), fe.reshape(-1, 3))
        if len(self.hinges):
            phi, sc, u = self._hinge(x[self.hinges])
            fe = (-self.hkb * sc * torch.sin((phi - self.phi0) / 2))[:, None, None] * u
            f = f.index_add(0, self.hinges.reshape(-1), fe.reshape(-1, 3))
        if self.contact_bodies:
            n, k = self.plane[:, :3], p["contact"][self.body]
            gap = (_dot(n, x) - self.plane[:, 3])[:, None]
            vn = _dot(n, v)[:, None]
            lam = -k[:, :1] * gap - k[:, 1:2] * vn
            ut = v - n * vn
            sp = (_dot(ut, ut)[:, None] + (gap >= 0)).sqrt()  # (not read off contact)
            lim = k[:, 3:] * lam.abs()
            ff = torch.where(k[:, 2:3] * sp <= lim, -k[:, 2:3] * ut, -lim * ut / sp)
            f = f + torch.where(self.on & (gap < 0), n * lam + ff, torch.zeros_like(f))
        v = v + (f / p["mass"][:, None] + self.g) * self.free * self.dt
        return x + v * self.dt, v

    def rollout(self, x, v, p, T, act=None):
        """T steps, checkpointed so that the tape of one segment is held at a time."""
        every = max(1, math.isqrt(T))

        def segment(x, v, t0, t1):
            for t in range(t0, t1):
                x, v = self.step(x, v, p, None if act is None else act[t])
            return x, v
        for t0 in range(0, T, every):
            x, v = checkpoint(segment, x, v, t0, min(T, t0 + every), use_reentrant=False)
        return x, v

    def mean_squared(self, x, target, nb):
        d = _dot(x - target, x - target)
        one = torch.zeros(nb, dtype=x.dtype, device=x.device).index_add(0, self.body, torch.ones_like(d))
        return torch.zeros_like(one).index_add(0, self.body, d) / one


def _params(bodies, grad):
    cat = lambda k: _t(np.concatenate([getattr(b, k) for b in bodies if getattr(b, k) is not None]))  # noqa: E731
    p = {"mass": cat("mass"), "contact": _t([[b.ke, b.kd, b.kf, b.muf] for b in bodies])}
    if any(b.ne for b in bodies):
        p["mu"], p["lam"] = cat("mu"), cat("lam")
    if any(b.nt for b in bodies):
        p["ktri"] = cat("ktri")
    if grad:
        for t in p.values():
            t.requires_grad_(True)
    if any(b.air for b in bodies):
        p["air"] = _t([[b.kdrag, b.klift] for b in bodies])
    return p


def _gradient(bodies, T, act=None):
    """(loss per body, xT, vT, d sum(loss) / d {x0, v0, parameters}) of a rollout."""
    ref, p = _Reference(bodies), _params(bodies, True)
    x0, v0 = (_t(np.concatenate([getattr(b, k) for b in bodies])).requires_grad_(True) for k in ("x0", "v0"))
    xT, vT = ref.rollout(x0, v0, p, T, act)
    loss = ref.mean_squared(xT, _t(np.concatenate([b.target for b in bodies])), len(bodies))
    loss.sum().backward()
    zero = lambda t: torch.zeros_like(t) if t.grad is None else t.grad
    g = {k: zero(t) for k, t in p.items() if t.requires_grad}
    g["mass"] = g["mass"] * ref.free[:, 0]
    return loss.detach(), xT.detach(), vT.detach(), dict(g, x0=zero(x0), v0=zero(v0))


def _soa(t):
    return t.detach().T.contiguous()


def _exact_rigid(case, seed):
    bodies, target = _rigid_bodies(case, seed)
    nb, nv = len(bodies), max(b.nv for b in bodies)
    V, Tg, live = np.zeros((nb, nv, 3)), np.zeros((nb, nv, 3)), np.zeros((nb, nv, 1))
    o = 0
    for i, b in enumerate(bodies):
        V[i, :b.nv], Tg[i, :b.nv], live[i, :b.nv] = b.verts, target[o:o + b.nv], 1
        o += b.nv
    V, Tg, live = _t(V), _t(Tg), _t(live)
    mass, inertia, contact, s0 = (_t(a).requires_grad_(True) for a in (
        [b.mass for b in bodies], [b.inertia for b in bodies], [b.contact() for b in bodies], [b.s0 for b in bodies]))
    plane, g, dt = _t([b.plane for b in bodies]), _t([b.gravity for b in bodies]), _t([[b.dt] for b in bodies])
    n, on = plane[:, None, :3], _t([[[float(b.ground)]] for b in bodies]) * live

    def rotation(q):
        w, a, b, c = q.unbind(1)
        return torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                            2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                            2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)], 1).view(-1, 3, 3)

    def apply(M, v):  # M [nb, 3, 3] on v [nb, ..., 3]
        return (M.view(nb, *([1] * (v.dim() - 2)), 3, 3) * v[..., None, :]).sum(-1)

    def mul(A, B):
        return (A[:, :, :, None] * B[:, None, :, :]).sum(2)

    def step(s):
        x, q, v, om = s[:, :3], s[:, 3:7], s[:, 7:10], s[:, 10:]
        R = rotation(q)
        a = apply(R, V)
        y, w = x[:, None] + a, v[:, None] + _cross(om[:, None].expand_as(a), a)
        k = contact[:, None]
        gap = (_dot(n.expand_as(y), y) - plane[:, None, 3])[..., None]
        vn = _dot(n.expand_as(w), w)[..., None]
        lam = -k[..., :1] * gap - k[..., 1:2] * vn
        ut = w - n * vn
        sp = (_dot(ut, ut)[..., None] + (gap >= 0)).sqrt()
        lim = k[..., 3:] * lam.abs()
        ff = torch.where(k[..., 2:3] * sp <= lim, -k[..., 2:3] * ut, -lim * ut / sp)
        f = torch.where((on > 0) & (gap < 0), n * lam + ff, torch.zeros_like(a))
        F, tau = f.sum(1), _cross(a, f).sum(1)
        i = inertia
        Ib = torch.stack([i[:, 0], i[:, 3], i[:, 4], i[:, 3], i[:, 1], i[:, 5], i[:, 4], i[:, 5], i[:, 2]], 1)
        Iw = mul(mul(R, Ib.view(-1, 3, 3)), R.transpose(1, 2))
        c = [_cross(Iw[:, 1], Iw[:, 2]), _cross(Iw[:, 2], Iw[:, 0]), _cross(Iw[:, 0], Iw[:, 1])]
        inv = torch.stack(c, 2) / _dot(Iw[:, 0], c[0])[:, None, None]
        om = om + dt * apply(inv, tau - _cross(om, apply(Iw, om)))
        v = v + dt * (F / mass[:, None] + g)
        u = q[:, 1:]
        q = torch.cat([q[:, :1] - dt / 2 * _dot(om, u)[:, None], u + dt / 2 * (om * q[:, :1] + _cross(om, u))], 1)
        return torch.cat([x + dt * v, q / _dot(q, q).sqrt()[:, None], v, om], 1)

    def segment(s, count):
        for _ in range(count):
            s = step(s)
        return s
    s, left, every = s0, case["steps"], max(1, math.isqrt(case["steps"]))
    while left:
        s = checkpoint(segment, s, min(left, every), use_reentrant=False)
        left -= min(left, every)
    d = (s[:, None, :3] + apply(rotation(s[:, 3:7]), V) - Tg) * live
    loss = (d * d).sum((1, 2)) / live.sum((1, 2))
    loss.sum().backward()
    return {"final": s.detach(), "loss": loss.detach(), "s0": s0.grad, "mass": mass.grad, "inertia": inertia.grad,
            "contact": contact.grad}


def _exact_silhouette(case, seed):
    tris, x, P, sigma, ibar = _view(case, seed)
    H, Wd = case["height"], case["width"]
    x, P = _t(x).requires_grad_(True), _t(P)
    hom = P[:, :3, None] * x[None]
    hom = hom.sum(1) + P[:, 3:]
    uv = (hom[:2] / hom[2]).T
    corners = uv.detach()[_t(tris, torch.int64)].requires_grad_(True)  # [nt, 3, 2]
    r = math.sqrt(13.815510557964274 * sigma)
    lo = torch.ceil(corners.detach().amin(1) - r - 0.5)
    size = torch.floor(corners.detach().amax(1) + r - 0.5) - lo + 1
    win = size.amax(0).long().tolist()

    def terms(c, lo):
        """Pixel index and softplus of the signed scaled distance over each triangle's window."""
        ox = torch.arange(win[0], device=c.device, dtype=torch.float64)
        oy = torch.arange(win[1], device=c.device, dtype=torch.float64)
        px = (lo[:, 0, None, None] + ox[None, None, :]).expand(len(c), win[1], win[0])
        py = (lo[:, 1, None, None] + oy[None, :, None]).expand(len(c), win[1], win[0])
        p = torch.stack([px, py], -1) + 0.5
        d2, side = [], []
        for a, b in ((0, 1), (1, 2), (2, 0)):
            A, B = c[:, a, None, None], c[:, b, None, None]
            e, w = B - A, p - A
            t = (_dot(w, e) / _dot(e, e)).clamp(0.0, 1.0)
            q = w - t[..., None] * e
            d2.append(_dot(q, q))
            side.append(e[..., 0] * w[..., 1] - e[..., 1] * w[..., 0])
        d = torch.minimum(torch.minimum(d2[0], d2[1]), d2[2])
        area = side[0] + side[1] + side[2]
        inside = (side[0] * area.sign() >= 0) & (side[1] * area.sign() >= 0) & (side[2] * area.sign() >= 0)
        keep = (inside | (d <= r * r)) & (px >= 0) & (px < Wd) & (py >= 0) & (py < H)
        z = torch.nn.functional.softplus(torch.where(inside, d, -d) / sigma, threshold=1e3)
        idx = (py.clamp(0, H - 1) * Wd + px.clamp(0, Wd - 1)).long()
        return idx, torch.where(keep, z, torch.zeros_like(z))
    chunk = max(1, 4_000_000 // (win[0] * win[1]))
    S = torch.zeros(H * Wd, dtype=torch.float64, device=x.device)
    with torch.no_grad():
        for i in range(0, len(corners), chunk):
            idx, z = terms(corners[i:i + chunk], lo[i:i + chunk])
            S.index_add_(0, idx.reshape(-1), z.reshape(-1))
    trans = torch.exp(-S)
    weight = _t(ibar).reshape(-1) * trans
    for i in range(0, len(corners), chunk):
        idx, z = terms(corners[i:i + chunk], lo[i:i + chunk])
        (weight[idx] * z).sum().backward()
    (uv[_t(tris, torch.int64)] * corners.grad).sum().backward()
    return {"image": (1 - trans).view(H, Wd), "x": x.grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "silhouette":
        return _exact_silhouette(case, seed)
    if kind == "rigid":
        return _exact_rigid(case, seed)
    if kind == "serve":
        out = []
        for b, t in _queries(case, seed):
            loss, _, _, g = _gradient([b], t)
            d = {"loss": float(loss[0]), "mass": g["mass"].cpu().numpy(), "contact": g["contact"].cpu().numpy()[0]}
            if b.ne:
                d.update(mu=g["mu"].cpu().numpy(), lam=g["lam"].cpu().numpy())
            if b.nt:
                d.update(k_tri=g["ktri"].cpu().numpy())
            out.append(d)
        return out
    bodies, T = _bodies(case, seed), case["steps"]
    if kind in ("step", "rollout"):
        with torch.no_grad():
            ref = _Reference(bodies)
            x, v = (_t(np.concatenate([getattr(b, k) for b in bodies])) for k in ("x0", "v0"))
            p = _params(bodies, False)
            for _ in range(T):
                x, v = ref.step(x, v, p, None)
        return _soa(x), _soa(v)
    act = w = None
    if kind == "control":
        w = _t(_weights(case, bodies, seed)).requires_grad_(True)
        tau = torch.arange(T, device=w.device, dtype=torch.float64)[:, None] * bodies[0].dt * OMEGA
        phase = torch.arange(SIGNALS, device=w.device, dtype=torch.float64)[None] * (2 * math.pi / SIGNALS)
        act = ACT_SCALE * torch.tanh((torch.sin(tau + phase)[:, :, None] * w[None]).sum(1))
    loss, x, v, g = _gradient(bodies, T, act)
    g["x0"], g["v0"] = g["x0"].T.contiguous(), g["v0"].T.contiguous()
    if case.get("via") == "autograd":  # one body: the mean over its particles
        keys = sorted(k for k in g if k not in ("x0", "v0"))
        return [loss[0], _soa(x), _soa(v), *(g[k] for k in keys), g["x0"], g["v0"]]
    out = {"loss": loss, "x": _soa(x), "v": _soa(v), **g}
    if kind == "control":
        out["W"] = w.grad
    return out
