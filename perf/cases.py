"""Timed cases of the step library: what programs built on it have it do.

A case is a dict of plain values.  `listed()` gives the fixed cases, `draw(rng)` one more of the
same ranges, `prepare(case, seed)` what a program holds before the call (a batch, a network or a
renderer with its inputs on the GPU), `run(state)` one pass through the public binding, `work(case)`
the bytes and operations a pass cannot do without, `exact(case, seed)` the outputs in 64 bits where
they are a plain function of the inputs.

Kinds of case
  step     flash_step with the exact contact metric (every contact solve to the tolerance)
  lite     flash_step in the fixed-budget mode (lightweight metric), from global memory
  forward  the warm-start network's forward pass
  grad     loss and gradient of one minibatch without allocation
  train    one epoch of the network trainer
  render   one frame of batched depth rendering
"""
import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2604_17513_amd import flash as F
from paper_2604_17513_amd import scenes

LAYERS = ((128, 16), (128, 128), (128, 128), (3, 128))   # (outputs, inputs) of W1..W4


def listed():
    return [
        # one FP64 env, default options: the smallest call a program makes (a cube at touchdown)
        dict(name="cube_1_fp64", kind="step", scene="cube", envs=1, size=4, K=20, fp64=True, fused=False, graph=False,
             groups=0, learned=False, reset=True, steps=2),
        # a small evaluation batch of distinct materials with the default options (one launch per phase)
        dict(name="squeeze_48", kind="step", scene="squeeze", envs=48, size=10, K=20, materials=48, fp64=False,
             fused=False, graph=False, groups=0, learned=False, reset=False, steps=1),
        # the benchmark's batch and launch configuration: 1024 envs, the local-global loop in one launch
        dict(name="squeeze_1024_fused", kind="step", scene="squeeze", envs=1024, size=10, K=20, materials=48,
             fp64=False, fused=True, graph=False, groups=0, learned=False, reset=False, steps=1),
        # sheets and blocks of uneven, odd sizes landing after a reset, on stream groups with graphs
        dict(name="uneven_96_groups", kind="step", scene="uneven", envs=96, sizes=7, size=17, vmax=1200, K=10, fp64=False,
             fused=True, graph=True, groups=3, learned=False, reset=True, steps=1),
        # FP64 sheets draping over a box from a reset (episode starts: cold multipliers)
        dict(name="cloth_64_fp64", kind="step", scene="cloth", envs=64, size=13, K=10, fp64=True, fused=True,
             graph=False, groups=0, learned=False, reset=True, steps=3),
        # fixed-budget folding of one garment-sized sheet: a chain of small launches
        dict(name="fold_1", kind="lite", scene="fold", envs=1, size=64, K=5, N=10, steps=1),
        # the same at a throughput batch: 256 copies share one inverse
        dict(name="fold_256", kind="lite", scene="fold", envs=256, size=64, K=5, N=10, steps=1),
        # fixed-budget mode over distinct sheets and blocks, each with an inverse of its own
        dict(name="uneven_lite_40", kind="lite", scene="uneven", envs=40, sizes=7, size=40, vmax=1800, K=10, N=10,
             reset=True, steps=1),
        # inference of the warm-start network over a rollout's contacts
        dict(name="forward_1m", kind="forward", rows=1048576),
        # one epoch of training, minibatches of 4096
        dict(name="train_64k", kind="train", rows=65536, batch=4096),
        # one camera frame for a single env: refit and rays of one surface
        dict(name="render_1", kind="render", mesh="towel", envs=1, size=181, width=128, height=128, points=True),
        # frames for a batch at camera resolution
        dict(name="render_48", kind="render", mesh="towel", envs=48, size=181, width=640, height=480, points=False),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "lite", "lite", "forward", "grad", "train", "render"])
    if kind == "step":
        scene = rng.choice(["cube", "squeeze", "squeeze", "uneven", "cloth"])
        c = dict(kind="step", scene=scene, fp64=rng.random() < 0.3, fused=rng.random() < 0.6, graph=rng.random() < 0.4,
                 groups=rng.choice([0, 0, 2, 3]), learned=rng.random() < 0.25, reset=True, K=20, steps=1)
        if scene == "cube":
            c.update(envs=_logint(rng, 1, 300), size=rng.randint(2, 6), steps=rng.randint(1, 2))
        elif scene == "squeeze":
            c.update(envs=_logint(rng, 2, 400), size=rng.randint(4, 10), materials=rng.randint(1, 32), reset=rng.random() < 0.3)
        elif scene == "uneven":
            c.update(envs=_logint(rng, 4, 96), sizes=rng.randint(0, 10 ** 6), size=17, vmax=1200, K=10)
        else:
            c.update(envs=_logint(rng, 1, 200), size=rng.randint(6, 17), K=10, steps=rng.randint(1, 3))
        c["groups"] = min(c["groups"], c["envs"]) if c["envs"] > 1 else 0
        return c
    if kind == "lite":
        K, N = rng.choice([(5, 10), (2, 2)])
        if rng.random() < 0.6:
            return dict(kind="lite", scene="fold", envs=_logint(rng, 1, 200), size=rng.randint(20, 64), K=K, N=N, steps=1)
        return dict(kind="lite", scene="uneven", envs=_logint(rng, 2, 32), sizes=rng.randint(0, 10 ** 6),
                    size=rng.randint(20, 40), vmax=rng.randint(700, 1800), K=2 * K, N=N,
                    reset=True, steps=1)
    if kind == "forward":
        return dict(kind="forward", rows=_logint(rng, 1, 4000000))
    if kind == "grad":
        return dict(kind="grad", rows=_logint(rng, 5, 2048))
    if kind == "train":
        batch = _logint(rng, 256, 8192)
        return dict(kind="train", rows=batch * rng.randint(1, 16) + rng.randint(0, batch - 1), batch=batch)
    w, h = rng.choice([(128, 128), (640, 480), (97, 65), (320, 240)])
    return dict(kind="render", mesh=rng.choice(["towel", "block"]), envs=_logint(rng, 1, 48),
                size=rng.randint(12, 181), width=w, height=h, points=rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------

def _cubes(case, seed):
    """Cubes half a millimetre above the ground at the end of a 0.2 m fall, jittered per env."""
    sc = scenes.drop_cube(seed=seed, hexes=case["size"], drop_height=5e-4, jitter=2e-4, lg_iterations=case["K"])
    rng = np.random.default_rng(seed)
    n = case["envs"]
    rest = sc.envs[0].rest_x
    sc.envs = sc.envs * n
    sc.x0 = [rest + np.array([0.0, 5e-4, 0.0]) + rng.uniform(-2e-4, 2e-4, size=rest.shape) for _ in range(n)]
    sc.v0 = [np.zeros_like(rest) + np.array([0.0, -1.98, 0.0]) for _ in range(n)]
    sc.obstacles = sc.obstacles * n
    return sc


def _squeeze(case, seed):
    """The benchmark's squeeze (closing for 64 steps); `materials` distinct (E, nu) over the envs, friction
    of each env its own."""
    sc = scenes.squeeze_blocks(case["envs"], seed=seed, hexes=case["size"], lg_iterations=case["K"],
                               close_speed=0.015, indent=1.5e-2)
    m = case["materials"]
    for e in range(m, case["envs"]):
        sc.envs[e].young, sc.envs[e].poisson = sc.envs[e % m].young, sc.envs[e % m].poisson
    return sc


def _cloths(case, seed):
    """Copies of one sheet just above a box, each with its own vertical jitter, falling at 0.5 m/s."""
    sc = scenes.cloth_drop(n=case["size"], height=2e-3, seed=seed, lg_iterations=case["K"])
    rng = np.random.default_rng(seed)
    n, nv = case["envs"], case["size"] ** 2
    base = sc.x0[0].copy()
    xs = []
    for _ in range(n):
        x = base.copy()
        x[:, 1] += rng.uniform(-1e-4, 1e-4, size=nv)
        xs.append(x)
    sc.envs, sc.x0, sc.obstacles = sc.envs * n, xs, sc.obstacles * n
    sc.v0 = [np.zeros_like(base) + np.array([0.0, -0.5, 0.0]) for _ in range(n)]
    return sc


def _folds(case, seed):
    """The folding sheet, each copy's rest height jittered by a few micrometres."""
    sc = scenes.cloth_fold(case["envs"], n=case["size"], lg_iterations=case["K"], inner_iterations=case["N"])
    rng = np.random.default_rng(seed)
    for x in sc.x0:
        x[:, 1] += rng.uniform(0.0, 1e-5, size=x.shape[0])
    return sc


@functools.lru_cache(maxsize=4)
def _uneven_bodies(envs, sizes, vmax, size, K):
    return scenes.uneven_batch(envs, seed=sizes, max_tet_vertices=vmax, max_cloth_side=size, lg_iterations=K)


def _uneven(case, seed):
    """The uneven recipe at touchdown: the case fixes the bodies' sizes and the obstacles' shapes, the
    seed their materials, positions and velocities.  Blocks also slide; obstacles hold."""
    base = _uneven_bodies(case["envs"], case["sizes"], case["vmax"], case["size"], case["K"])
    rng = np.random.default_rng(seed)
    envs, xs, vs, obs = [], [], [], []
    for e, env in enumerate(base.envs):
        sheet = env.elem == scenes.TRI
        drop, slide = (0.0485, 0.0) if sheet else (0.001, 0.3)
        envs.append(dataclasses.replace(env, young=env.young * float(rng.uniform(0.8, 1.25)), mu=float(rng.uniform(0.3, 0.8))))
        xs.append(base.x0[e] - np.array([0.0, drop, 0.0]))
        vs.append(np.zeros_like(xs[-1]) + np.array([rng.uniform(-slide, slide), -rng.uniform(0.3, 1.0),
                                                    rng.uniform(-slide, slide)]))
        lst = [o.copy() for o in base.obstacles[e]]
        for o in lst[1:]:
            o.center = o.center + np.array([rng.uniform(-0.02, 0.02), -drop, rng.uniform(-0.02, 0.02)])
            o.move_steps = 0
        obs.append(lst)
    params = dataclasses.replace(base.params)
    if case["kind"] == "lite":
        params.max_inner_iterations = case["N"]
    return scenes.Scene(envs, xs, vs, obs, params, name="uneven")


def _scene(case, seed):
    if case["scene"] == "cube":
        return _cubes(case, seed)
    if case["scene"] == "squeeze":
        return _squeeze(case, seed)
    if case["scene"] == "cloth":
        return _cloths(case, seed)
    if case["scene"] == "fold":
        return _folds(case, seed)
    return _uneven(case, seed)


def _network(seed, rows):
    """A network and the normalisation of standardised features (the bias column passes through)."""
    m = F.Mlp(max(rows, 64), seed=seed % 1000003)
    norm = np.zeros(F.MLP_NORM, dtype=np.float32)
    norm[16:] = 1.0
    norm[15], norm[31] = 0.0, 1.0
    m.set_norm(norm)
    return m


def _features(rows, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn((rows, 16), generator=g, device="cuda", dtype=torch.float32)
    x[:, 15] = 1.0
    return x


def _targets(x, seed):
    """Labels of a fixed smooth map of the features plus noise."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    a = torch.randn((16, 3), generator=g, device="cuda", dtype=torch.float32) / 4.0
    return torch.tanh(x @ a) + 0.05 * torch.randn((x.shape[0], 3), generator=g, device="cuda", dtype=torch.float32)


def _surface(case):
    if case["mesh"] == "towel":
        rest, tris = scenes.cloth_grid(case["size"], 0.6, (-0.3, -0.3), 0.0)
        return scenes.EnvDesc(scenes.TRI, rest, tris)
    k = max(2, min(12, case["size"] // 8))
    rest, tets = scenes.hex_lattice(k, k, k, (0.3, 0.2, 0.3), (-0.15, 0.0, -0.15))
    return scenes.EnvDesc(scenes.TET, rest, tets)


def _views(case, seed):
    """Per-env surfaces in seeded folds over a table, and one top-down camera per env."""
    env = _surface(case)
    rng = np.random.default_rng(seed)
    xs = []
    for _ in range(case["envs"]):
        x = env.rest_x.copy()
        k, ph = rng.uniform(6.0, 14.0, size=2), rng.uniform(0.0, 2 * np.pi, size=2)
        x[:, 1] += 0.03 + 0.028 * np.sin(k[0] * env.rest_x[:, 0] + ph[0]) * np.cos(k[1] * env.rest_x[:, 2] + ph[1])
        xs.append(x)
    down = np.array([[1.0, 0.0, 0.0], [0.0, 0.0, -1.0], [0.0, 1.0, 0.0]])
    cam = {"position": np.array([0.013, 0.9, 0.007]), "rot": down, "fx": 0.78 * case["width"],
           "fy": 0.78 * case["width"], "cx": case["width"] / 2.0, "cy": case["height"] / 2.0}
    x = torch.tensor(np.concatenate(xs).T.copy(), dtype=torch.float32, device="cuda")
    return env, x, cam


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "lite"):
        sc = _scene(case, seed)
        if kind == "lite":
            cap = max(e.n_vertices for e in sc.envs) + 8 if case["scene"] == "fold" else 3000
            b = F.from_scene(sc, contact_metric=F.FLASH_METRIC_LIGHTWEIGHT, global_contact_solve=1, max_contacts=cap,
                             use_graph=True)
        else:
            b = F.from_scene(sc, precision=F.FLASH_FP64 if case["fp64"] else F.FLASH_FP32, use_graph=case["graph"],
                             stream_groups=case["groups"], fused_lg=case["fused"],
                             warm_start=F.FLASH_WS_LEARNED if case["learned"] else F.FLASH_WS_PREV)
            if case["learned"]:
                m = _network(seed, 64)
                b.ws_load(m.params_bf16(), m.norm())
        dt = torch.float64 if case.get("fp64") else torch.float32
        n = sum(b.nv)
        x, v = (torch.empty((3, n), dtype=dt, device="cuda") for _ in range(2))
        s = {"batch": b, "steps": case["steps"], "x": x, "v": v, "x0": None, "v0": None}
        if case["scene"] == "squeeze" and case["reset"]:
            # every pass drops the multiplier history, as episode resets do: the state is set to itself
            b.step(8)
            b.get_state_device(x, v)
            s["x0"], s["v0"] = x, v
        elif case.get("reset"):
            s["x0"], s["v0"] = (torch.tensor(np.concatenate(a).T.copy(), dtype=dt, device="cuda") for a in (sc.x0, sc.v0))
        else:
            b.step(8 if case["scene"] == "squeeze" else 4)
        b.synchronize()
        return s
    if kind == "forward":
        return {"net": _network(seed, 64), "x": _features(case["rows"], seed),
                "y": torch.empty((case["rows"], 3), dtype=torch.float32, device="cuda")}
    if kind == "grad":
        x = _features(case["rows"], seed)
        w = torch.tensor(_network(seed, 64).params(), device="cuda")
        return {"w": w, "x": x, "t": _targets(x, seed), "g": torch.empty(F.MLP_PARAMS, dtype=torch.float32, device="cuda"),
                "loss": torch.empty(1, dtype=torch.float32, device="cuda")}
    if kind == "train":
        x = _features(case["rows"], seed)
        return {"net": _network(seed, case["batch"]), "x": x, "t": _targets(x, seed), "batch": case["batch"]}
    env, x, cam = _views(case, seed)
    n = case["envs"]
    return {"renderer": F.Renderer([env] * n), "x": x, "cams": [cam] * n, "obs": [[scenes.ground()]] * n,
            "w": case["width"], "h": case["height"], "points": case["points"]}


def run(state):
    if "batch" in state and "steps" in state:
        b = state["batch"]
        if state["x0"] is not None:
            b.set_state_device(state["x0"], state["v0"])
        b.step(state["steps"])
        b.get_state_device(state["x"], state["v"])
        b.synchronize()   # the batch runs on a stream of its own: the program waits before it reads x and v
        return {"x": state["x"], "v": state["v"]}
    if "renderer" in state:
        return state["renderer"].render(state["x"], state["cams"], state["w"], state["h"], obstacles=state["obs"],
                                        points=state["points"])
    n = state["x"].shape[0]
    if "y" in state:
        state["net"].forward(state["x"], n, state["y"])
        return state["y"]
    if "g" in state:
        F.mlp_grad_noalloc(state["w"], state["x"], state["t"], n, state["g"], state["loss"],
                           stream=torch.cuda.current_stream().cuda_stream)
        return {"grad": state["g"], "loss": state["loss"]}
    losses = state["net"].train(state["x"], state["t"], n, 1, batch=state["batch"], lr=1e-3, seed=1)
    return {"losses": losses, "params": state["net"].params()}


# ---------------------------------------------------------------------------------------------
# least bytes and operations of a pass
# ---------------------------------------------------------------------------------------------

def _bodies(case):
    """(vertices, elements, contacts, envs sharing the inverse) of each distinct body: the lattices' own
    counts, and for the uneven recipe a fixed sample of its sizes."""
    k, n = case["size"], case["envs"]
    if case["scene"] == "cube":
        return [((k + 1) ** 3, 6 * k ** 3, (k + 1) ** 2, n)]
    if case["scene"] == "squeeze":
        m = min(case["materials"], n)
        return [((k + 1) ** 3, 6 * k ** 3, 1.8 * (k + 1) ** 2, n / m)] * m
    if case["scene"] == "cloth":
        return [(k * k, 2 * (k - 1) ** 2, 0.15 * k * k, n)]
    if case["scene"] == "fold":
        return [(k * k, 2 * (k - 1) ** 2, k * k - 8, n)]
    rng = np.random.default_rng(0)
    out = []
    for _ in range(n):
        if rng.random() < 0.5:
            side = int(round(np.exp(rng.uniform(np.log(16), np.log(max(k, 17))))))
            out.append((side * side, 2 * (side - 1) ** 2, side * side, 1))
        else:
            nv = np.exp(rng.uniform(np.log(500), np.log(case["vmax"])))
            out.append((nv, 5 * nv, nv ** (2.0 / 3.0), 1))
    return out


def work(case):
    kind = case["kind"]
    if kind in ("step", "lite"):
        fp = 8 if case.get("fp64") else 4
        by = fl = 0.0
        for nv, ne, nc, share in _bodies(case):
            tri = fp * nv * (nv + 1) / 2            # the symmetric inverse, once for the envs that share it
            per_lg = share * (14 * fp * ne + 9 * fp * nv) + tri
            fl_lg = share * (6 * nv * nv + 300 * ne)
            if kind == "lite":                      # N + 1 position updates over the contact rows
                upd = min(tri, fp * nc * nv)
                per_lg += (case["N"] + 1) * (upd + share * (9 * fp * nv + 27 * fp * nc))
                fl_lg += (case["N"] + 1) * share * (6 * nv * nc + 100 * nc)
            else:                                   # the position update and about half a Newton iteration
                per_lg += share * 27 * fp * nc
                fl_lg += share * (6 * nv * nc + 9 * nc * nc)
            by += case["K"] * per_lg + share * (18 * fp * nv + 16 * fp * nc)
            fl += case["K"] * fl_lg
        return {"bytes": case["steps"] * by, "flops": case["steps"] * fl}
    per_row = 2.0 * sum(o * i for o, i in LAYERS)
    if kind == "forward":
        return {"bytes": case["rows"] * 76.0 + 4 * F.MLP_PARAMS, "flops": case["rows"] * per_row}
    if kind == "grad":
        return {"bytes": case["rows"] * 76.0 + 8 * F.MLP_PARAMS, "flops": case["rows"] * 3 * per_row}
    if kind == "train":
        steps = case["rows"] // case["batch"]
        return {"bytes": steps * (case["batch"] * 76.0 + 28 * F.MLP_PARAMS),
                "flops": steps * case["batch"] * 3 * per_row}
    env = _surface(case)
    px = case["envs"] * case["width"] * case["height"]
    tris = 2 * (case["size"] - 1) ** 2 if case["mesh"] == "towel" else 12 * (max(2, min(12, case["size"] // 8))) ** 2
    out = 8 + (12 if case["points"] else 0)
    return {"bytes": float(px * out + case["envs"] * 12 * env.n_vertices),
            "flops": float(px * (40 * math.log2(tris) + 200) + case["envs"] * 30 * tris)}


# ---------------------------------------------------------------------------------------------
# outputs in 64 bits
# ---------------------------------------------------------------------------------------------

def _layers64(w):
    out, o = [], 0
    for no, ni in LAYERS:
        W = w[o:o + no * ni].reshape(no, ni)
        b = w[o + no * ni:o + no * ni + no]
        out.append((W, b))
        o += no * ni + no
    return out


def exact(case, seed):
    """The network's outputs and gradients in 64 bits; a single env's small image by casting every ray
    against every triangle in 64 bits.  A step's contact solves stop at a tolerance or after a fixed
    number of updates, and training rounds its operands in every minibatch: their states have no value
    that a formula gives."""
    kind = case["kind"]
    if kind in ("forward", "grad"):
        s = prepare(case, seed)
        w = (s["w"].double() if "w" in s else torch.tensor(s["net"].params(), device="cuda").double()).requires_grad_(kind == "grad")
        h = s["x"].double()
        for i, (W, b) in enumerate(_layers64(w)):
            h = h @ W.T + b
            if i < 3:
                h = torch.relu(h)
        if kind == "forward":
            return h
        loss = ((h - s["t"].double()) ** 2).mean()
        loss.backward()
        return {"grad": w.grad, "loss": loss.detach().reshape(1)}
    if kind != "render" or case["envs"] * case["width"] * case["height"] > 20000:
        return None
    env, x, cam = _views(case, seed)
    if env.elem != scenes.TRI:
        return None
    X = x.double()
    tri = torch.tensor(env.elements.astype(np.int64), device="cuda")
    dep, pts = [], []
    W, H = case["width"], case["height"]
    v, u = torch.meshgrid(torch.arange(H, device="cuda"), torch.arange(W, device="cuda"), indexing="ij")
    R = torch.tensor(cam["rot"], device="cuda", dtype=torch.float64)
    o = torch.tensor(cam["position"], device="cuda", dtype=torch.float64)
    u, v = u.double(), v.double()
    ray = torch.stack([(u + 0.5 - cam["cx"]) / cam["fx"], (v + 0.5 - cam["cy"]) / cam["fy"], torch.ones_like(u)], -1)
    D = ray.reshape(-1, 3) @ R.T
    for e in range(case["envs"]):
        P = X[:, e * env.n_vertices:(e + 1) * env.n_vertices].T
        A, B, C = (P[tri[:, k]] for k in range(3))
        e1, e2, s = B - A, C - A, o - A
        q = torch.linalg.cross(s, e1)
        n = torch.linalg.cross(e1, e2)
        se = torch.linalg.cross(s, e2)
        t = torch.full((D.shape[0],), math.inf, dtype=torch.float64, device="cuda")
        for r0 in range(0, D.shape[0], 256):
            d = D[r0:r0 + 256]
            det = -(d @ n.T)                         # (d x e2) . e1
            b1 = -(d @ se.T) / det                   # (d x e2) . s
            b2 = (d @ q.T) / det
            th = (e2 * q).sum(-1)[None] / det
            hit = (b1 >= 0) & (b2 >= 0) & (b1 + b2 <= 1) & (th > 0)
            t[r0:r0 + 256] = torch.where(hit, th, math.inf).min(1).values
        tg = -o[1] / D[:, 1]                         # the table plane y = 0
        t = torch.minimum(t, torch.where(tg > 0, tg, math.inf))
        ok = torch.isfinite(t)
        dep.append(torch.where(ok, t, 0.0).reshape(H, W))
        pts.append(torch.where(ok[:, None], o + t[:, None] * D, 0.0).reshape(H, W, 3))
    out = {"depth": torch.stack(dep), "instance": None}
    if case["points"]:
        out["points"] = torch.stack(pts)
    return out
