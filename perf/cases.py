"""The work that programs have this framework do, as cases that can be timed.

Every case goes through the public entry points (``paper_2207_09334_amd.cronos``) the way the
framework's own drivers do: a simulation handle is created once and then stepped and read
frame by frame; a population handle is kept and every rollout resets it to the rest state under
another actuation; a gait gradient resets, rolls out and sweeps back; natural frequencies are
asked of a body as it stands; the surrogate network is trained on minibatches and screens rows
of candidates.

State that the device holds in FP32 (positions, velocities, forces, gradients, parameters) is
returned in FP32; the library's FP64 results (natural frequencies) in FP64.

``exact`` computes the same outputs in FP64 with plain torch and numpy from the same inputs.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2207_09334_amd import cronos as CR

GRAVITY = (0.0, 0.0, -9.81)
MATERIAL_K = (1.0e3, 1.0e4, 1.0e5)
NET_IN, NET_OUT = 96, 3
CORNERS = np.array([[i & 1, (i >> 1) & 1, i >> 2] for i in range(8)], np.int64)


# ------------------------------------------------------------------------------ the cases

def listed():
    return [
        # An interactive program's frame of the smallest body: a few steps, then its state.
        {"name": "cube_frame", "kind": "frame", "body": "cube", "nx": 10, "ny": 10, "nz": 10, "steps": 10},
        # A drop of the same body in the one-workgroup form: many steps a call.
        {"name": "cube_resident", "kind": "frame", "body": "cube", "nx": 10, "ny": 10, "nz": 10, "steps": 400,
         "resident": True},
        # The actuated legged robot on the ground, one frame of 10 ms.
        {"name": "quadruped_frame", "kind": "frame", "body": "quadruped", "steps": 100},
        # A beam whose sides are no multiple of anything (general entries), Verlet integrator.
        {"name": "beam_ragged_verlet", "kind": "frame", "body": "beam", "nx": 121, "ny": 27, "nz": 19, "steps": 200,
         "verlet": True},
        # The headline cantilever: a full box of 640,000 masses, 50 ms of motion.
        {"name": "cantilever_640k", "kind": "frame", "body": "beam", "nx": 400, "ny": 40, "nz": 40, "steps": 1000},
        # A quasi-uniform point lattice (each spring its own stiffness and length).
        {"name": "point_bar", "kind": "frame", "body": "points", "nx": 100, "ny": 22, "nz": 22, "steps": 200},
        # A population of random-walk robots: reset, new actuation, roll out, read.
        {"name": "population_rollout", "kind": "population", "robots": 64, "hi": 20000, "steps": 1000},
        # The gait gradient of the quadruped: reset, rollout with checkpoints, reverse sweep.
        {"name": "gait_gradient", "kind": "gait", "steps": 200, "ckpt": 50},
        # Lowest frequencies of a small and of a large beam.
        {"name": "frequencies_small", "kind": "modes", "nx": 48, "ny": 20, "nz": 12, "modes": 2},
        {"name": "frequencies_large", "kind": "modes", "nx": 128, "ny": 40, "nz": 32, "modes": 2},
        # Surrogate training: epochs over rollouts in minibatches of 1024.
        {"name": "surrogate_train", "kind": "train", "rows": 8192, "width": 768, "batch": 1024, "epochs": 2},
        # Surrogate screening of a pool's candidates.
        {"name": "surrogate_screen", "kind": "screen", "rows": 16384, "width": 768, "max_rows": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed kinds; sizes log-uniform, odd ones as likely as even ones."""
    kind = rng.choice(["cube", "resident", "quadruped", "beam", "box", "points", "population", "gait", "modes",
                       "train", "screen", "inspect", "gradient"])
    if kind == "cube":
        return {"kind": "frame", "body": "cube", "nx": _log(rng, 2, 40), "ny": _log(rng, 2, 40),
                "nz": _log(rng, 2, 40), "steps": _log(rng, 1, 200)}
    if kind == "resident":
        n = rng.randint(3, 10)
        return {"kind": "frame", "body": "cube", "nx": n, "ny": rng.randint(3, 10), "nz": n,
                "steps": _log(rng, 10, 400), "resident": True}
    if kind == "quadruped":
        return {"kind": "frame", "body": "quadruped", "steps": _log(rng, 1, 250)}
    if kind == "beam":
        return {"kind": "frame", "body": "beam", "nx": _log(rng, 20, 300), "ny": _log(rng, 5, 41),
                "nz": _log(rng, 5, 41), "steps": _log(rng, 20, 400), "verlet": rng.random() < 0.5}
    if kind == "box":
        return {"kind": "frame", "body": "beam", "nx": 8 * rng.randint(16, 50), "ny": 8 * rng.randint(4, 5),
                "nz": 8 * rng.randint(4, 5), "steps": _log(rng, 20, 800), "verlet": rng.random() < 0.5}
    if kind == "points":
        return {"kind": "frame", "body": "points", "nx": _log(rng, 10, 150), "ny": _log(rng, 5, 24),
                "nz": _log(rng, 5, 24), "steps": _log(rng, 10, 300)}
    if kind == "population":
        return {"kind": "population", "robots": _log(rng, 2, 64), "hi": _log(rng, 1000, 20000),
                "steps": _log(rng, 100, 800)}
    if kind == "gait":
        return {"kind": "gait", "steps": _log(rng, 20, 200), "ckpt": _log(rng, 10, 100)}
    if kind == "modes":
        # sides apart from each other: bending in y and in z must not share one frequency
        nz = rng.randint(6, 20)
        return {"kind": "modes", "nx": nz + rng.randint(20, 60), "ny": nz + rng.randint(6, 14), "nz": nz,
                "modes": rng.randint(1, 3)}
    if kind == "train":
        rows = _log(rng, 500, 12000)
        return {"kind": "train", "rows": rows, "width": rng.choice([64, 200, 256, 512, 768]),
                "batch": min(rows, rng.choice([128, 500, 1024])), "epochs": 1}
    if kind == "screen":
        return {"kind": "screen", "rows": _log(rng, 1, 20000), "width": rng.choice([256, 768]),
                "max_rows": rng.choice([512, 1024, 4096])}
    if kind == "gradient":
        return {"kind": "gradient", "rows": _log(rng, 1, 4096), "width": rng.choice([256, 768])}
    return {"kind": "inspect", "body": "beam", "nx": _log(rng, 8, 250), "ny": _log(rng, 5, 41),
            "nz": _log(rng, 5, 41)}


# ------------------------------------------------------------------------------ bodies (plain numpy)

def _voxel_lattice(voxels, material_k, material, group, spacing):
    """Nodes and springs of one body's voxels: corners in (z, y, x) order, every pair of a voxel's
    corners linked, stiffness summed over the voxels that hold the link (a quarter, a half or all
    of the voxel's for an edge, a face or a body diagonal), the actuation group of the first
    actuated voxel in (z, y, x) order that holds it."""
    vox = np.asarray(voxels, np.int64)
    order = np.lexsort((vox[:, 0], vox[:, 1], vox[:, 2]))
    vox, mat = vox[order], np.asarray(material)[order]
    grp = np.full(len(vox), -1) if group is None else np.asarray(group)[order]
    corner = vox[:, None, :] + CORNERS[None]
    key = (corner[..., 2] << 42) | (corner[..., 1] << 21) | corner[..., 0]
    nodes, inv = np.unique(key.ravel(), return_inverse=True)
    inv = inv.reshape(-1, 8)
    coords = np.stack([nodes & 0x1FFFFF, (nodes >> 21) & 0x1FFFFF, nodes >> 42], 1).astype(np.int32)
    a, b = np.triu_indices(8, 1)
    kind = (CORNERS[a] != CORNERS[b]).sum(1)
    lo, hi = np.minimum(inv[:, a], inv[:, b]).ravel(), np.maximum(inv[:, a], inv[:, b]).ravel()
    link, which = np.unique(lo.astype(np.int64) * len(nodes) + hi, return_inverse=True)
    which = which.ravel()
    weight = np.array([0.0, 0.25, 0.5, 1.0])[kind]
    k = np.bincount(which, (np.asarray(material_k)[mat][:, None] * weight[None]).ravel(), len(link))
    first = np.full(len(link), len(vox))
    holder = np.repeat(np.arange(len(vox)), len(a))
    np.minimum.at(first, which, np.where(grp[holder] >= 0, holder, len(vox)))
    g = np.where(first < len(vox), np.append(grp, -1)[np.minimum(first, len(vox))], -1).astype(np.int16)
    rest = np.empty(len(link))
    rest[which] = spacing * np.sqrt(np.tile(kind, len(vox)))
    ends = np.stack([link // len(nodes), link % len(nodes)], 1).astype(np.int32)
    return {"coords": coords, "x": spacing * coords.astype(float), "ends": ends, "k": k, "rest": rest, "group": g}


def _box_lattice(nx, ny, nz, voxel_k, spacing):
    """The same for a full box of nodes, direction by direction."""
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    coords = np.stack([x.ravel(), y.ravel(), z.ravel()], 1).astype(np.int32)
    index = np.arange(nx * ny * nz).reshape(nz, ny, nx)
    ends, k, rest = [], [], []
    for d in range(14, 27):
        o = (d % 3 - 1, d // 3 % 3 - 1, d // 9 - 1)
        cut = [(slice(max(0, -c), n - max(0, c)), slice(max(0, c), n - max(0, -c))) for c, n in zip(o, (nx, ny, nz))]
        i, j = (index[cut[2][e], cut[1][e], cut[0][e]].ravel() for e in (0, 1))
        # voxels that hold the link: one along each axis it spans, one or two (inside) along the others
        held = np.ones(len(i))
        for c, n in enumerate((nx, ny, nz)):
            if o[c] == 0:
                held *= np.where((coords[i, c] > 0) & (coords[i, c] < n - 1), 2.0, 1.0)
        kind = sum(c != 0 for c in o)
        ends.append(np.stack([i, j], 1))
        k.append(voxel_k * (0.0, 0.25, 0.5, 1.0)[kind] * held)
        rest.append(np.full(len(i), spacing * math.sqrt(kind)))
    corners = np.ones(len(coords))
    for c, n in enumerate((nx, ny, nz)):
        corners *= np.where((coords[:, c] > 0) & (coords[:, c] < n - 1), 2.0, 1.0)
    return {"coords": coords, "x": spacing * coords.astype(float), "ends": np.concatenate(ends).astype(np.int32),
            "k": np.concatenate(k), "rest": np.concatenate(rest), "corners": corners}


def _walk(rng, target):
    """Voxels of a random walk in order of first visit, until their corners number `target`."""
    steps = np.array([[1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1]], np.int64)
    pos = np.concatenate([np.zeros((1, 3), np.int64), np.cumsum(steps[rng.integers(0, 6, max(64, 4 * target))], 0)])
    pos -= pos.min(0)
    key = (pos[:, 2] << 42) | (pos[:, 1] << 21) | pos[:, 0]
    _, first = np.unique(key, return_index=True)
    vox = pos[np.sort(first)]
    corner = vox[:, None, :] + CORNERS[None]
    ck = ((corner[..., 2] << 42) | (corner[..., 1] << 21) | corner[..., 0]).ravel()
    _, at = np.unique(ck, return_index=True)
    count = np.cumsum(np.bincount(at // 8, minlength=len(vox)))
    vox = vox[:min(len(vox), int(np.searchsorted(count, target)) + 1)]
    return vox - vox.min(0)


def _stack(bodies):
    """Several bodies as one system."""
    base = np.cumsum([0] + [len(b["x"]) for b in bodies])
    out = {f: np.concatenate([b[f] for b in bodies]) for f in ("coords", "x", "k", "rest", "group")}
    out["ends"] = np.concatenate([b["ends"] + o for b, o in zip(bodies, base)]).astype(np.int32)
    out["body_offset"] = base.astype(np.int64)
    out["spring_body"] = np.repeat(np.arange(len(bodies)), [len(b["k"]) for b in bodies])
    return out


@functools.lru_cache(maxsize=2)
def _geometry(what):
    """What a program builds once: the body's nodes, springs and constants (no seeded input)."""
    case = dict(what)
    body = case.get("body") or {"population": "robots", "gait": "quadruped", "modes": "beam"}[case["kind"]]
    if body == "cube":
        g = _box_lattice(case["nx"], case["ny"], case["nz"], 1.0, 0.01)
        g.update(k=np.full(len(g["k"]), 1.0e4), mass=np.full(len(g["x"]), 1.0e-3), damping=0.01, dt=1.0e-4, ground=True,
                 x=g["x"] + np.array([0.0, 0.0, 0.002]), jitter=1.0e-4)
    elif body == "beam":
        a = 0.005
        g = _box_lattice(case["nx"], case["ny"], case["nz"], 1.0e6 * a / 2.7, a)
        g.update(mass=g["corners"] * 1000.0 * a ** 3 / 8.0, damping=0.0, dt=5.0e-5, ground=False,
                 pinned=(g["coords"][:, 0] == 0).astype(np.uint8), jitter=1.0e-5)
    elif body == "quadruped":
        box = lambda n, o: np.stack(np.meshgrid(*[np.arange(c) + s for c, s in zip(n, o)], indexing="ij"),
                                    -1).reshape(-1, 3)
        torso, legs = box((40, 20, 10), (0, 0, 10)), [box((8, 8, 10), (x, y, 0)) for x in (0, 32) for y in (0, 12)]
        region = [8 + torso[:, 1] // 10 * 4 + torso[:, 0] // 10] + [2 * q + (v[:, 2] >= 5) for q, v in enumerate(legs)]
        vox, region = np.concatenate([torso] + legs), np.concatenate(region)
        mat = np.random.default_rng(2).integers(0, 3, len(vox))
        g = _stack([_voxel_lattice(vox, MATERIAL_K, mat, np.where(mat < 2, region, -1), 0.01)])
        g.update(mass=np.full(len(g["x"]), 0.1), damping=1.0e-4, dt=1.0e-4, ground=True, n_groups=16, amp=(0.2, 0.2),
                 jitter=1.0e-6)
    elif body == "robots":
        rng, bodies = np.random.default_rng(3), []
        for _ in range(case["robots"]):
            vox = _walk(rng, int(round(math.exp(rng.uniform(math.log(500), math.log(case["hi"]))))))
            mat = rng.integers(0, 3, len(vox))
            bodies.append(_voxel_lattice(vox, MATERIAL_K, mat, np.where(mat < 2, np.arange(len(vox)) * 32 // len(vox), -1),
                                         0.01))
        g = _stack(bodies)
        g.update(mass=np.full(len(g["x"]), 0.1), damping=1.0e-4, dt=1.0e-4, ground=True, n_groups=32, amp=(0.0, 0.25),
                 jitter=0.0)
    else:  # points: a jittered grid, springs up to 1.6 mean spacings
        s, n = 0.0015, (case["nx"], case["ny"], case["nz"])
        z, y, x = np.meshgrid(*[np.arange(c) for c in n[::-1]], indexing="ij")
        pts = s * (np.stack([x, y, z], -1) + 0.5 + np.random.default_rng(5).uniform(-0.25, 0.25, x.shape + (3,)))
        index, ends = np.arange(pts.size // 3).reshape(x.shape), []
        for d in range(63, 125):
            o = (d % 5 - 2, d // 5 % 5 - 2, d // 25 - 2)
            if any(abs(c) >= m for c, m in zip(o, n)):
                continue
            cut = [(slice(max(0, -c), m - max(0, c)), slice(max(0, c), m - max(0, -c))) for c, m in zip(o, n)]
            i, j = (index[cut[2][e], cut[1][e], cut[0][e]].ravel() for e in (0, 1))
            near = np.linalg.norm(pts.reshape(-1, 3)[j] - pts.reshape(-1, 3)[i], axis=1) <= 1.6 * s
            ends.append(np.stack([i[near], j[near]], 1))
        pts, ends = pts.reshape(-1, 3), np.concatenate(ends).astype(np.int32)
        rest = np.linalg.norm(pts[ends[:, 1]] - pts[ends[:, 0]], axis=1)
        g = {"x": pts, "ends": ends, "rest": rest, "k": 1.0e4 * s / rest, "mass": np.full(len(pts), 0.1),
             "pinned": (pts[:, 0] < 0.75 * s).astype(np.uint8), "damping": 0.0, "dt": 1.0e-4, "ground": False,
             "jitter": 1.0e-6}
    if case["kind"] == "modes":
        g["jitter"] = 2.0e-4
    return g


def _of(case):
    keep = ("kind", "body", "nx", "ny", "nz", "robots", "hi")
    return _geometry(tuple((k, case[k]) for k in keep if k in case))


def _inputs(g, seed):
    """The seeded inputs: node jitter, a velocity along the body and the actuation."""
    rng = np.random.default_rng(seed)
    free = np.ones((len(g["x"]), 1)) if "pinned" not in g else 1.0 - g["pinned"][:, None]
    x0 = g["x"] + free * g["jitter"] * rng.uniform(-1.0, 1.0, g["x"].shape)
    along = g["x"][:, :1] / max(float(g["x"][:, 0].max()), 1e-9)
    v0 = free * along ** 2 * rng.uniform(-0.05, 0.05, (1, 3))
    count = g.get("n_groups", 0) * (len(g["body_offset"]) - 1 if "body_offset" in g else 1)
    phase, amp = 2.0 * math.pi * rng.random(count), rng.uniform(*g.get("amp", (0.0, 0.0)), count)
    return x0, v0, phase, amp


def _create(case, g, x0, v0, gravity=GRAVITY):
    groups = g.get("n_groups", 0)
    several = len(g.get("body_offset", ())) > 2
    flags = (CR.VERLET if case.get("verlet") else 0) | (CR.RESIDENT if case.get("resident") else 0)
    return CR.cronos_create(x0, g["mass"], g["ends"], g["k"], g["rest"], v0=v0, pinned=g.get("pinned"),
                            grid=g.get("coords"), group=g["group"] if groups else None, n_groups=groups,
                            body_offset=g["body_offset"] if several else None, gravity=gravity, damping=g["damping"],
                            dt=g["dt"], ground=g["ground"], ground_k=1.0e5 if g["ground"] else 0.0,
                            ground_mu=0.8 if g["ground"] else 0.0, flags=flags)


# one handle of a population or gait problem serves every rollout of it, as a screening or an
# optimising program keeps it; every pass resets it
_handles = {}


def _handle(case, g):
    key = tuple(sorted((k, v) for k, v in case.items() if k in ("kind", "robots", "hi")))
    if key not in _handles:
        if len(_handles) > 1:
            _handles.pop(next(iter(_handles)))["sim"].close()
        _handles[key] = {"sim": _create(case, g, g["x"], np.zeros_like(g["x"]))}
    return _handles[key]["sim"]


def _network(case, seed):
    rng = np.random.default_rng(seed)
    sizes = (NET_IN,) + (case["width"],) * 3 + (NET_OUT,)
    params = []
    for i, o in zip(sizes, sizes[1:]):
        params += [rng.uniform(-1.0, 1.0, (i, o)) * math.sqrt(6.0 / (i + o)), 0.05 * rng.normal(size=o)]
    X = rng.normal(size=(case["rows"], NET_IN)).astype(np.float32)
    T = np.tanh(X[:, :3] + 0.1 * X[:, 3:6] * X[:, 6:9]).astype(np.float32)
    return sizes, params, X, T


# ------------------------------------------------------------------------------ a pass

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("train", "screen", "gradient"):
        sizes, params, X, T = _network(case, seed)
        rows = case["batch"] if kind == "train" else case.get("max_rows", case["rows"])
        return {"case": case, "net": CR.cronos_mlp_create(params, sizes=sizes, max_rows=rows), "X": X, "T": T}
    g = _of(case)
    x0, v0, phase, amp = _inputs(g, seed)
    if kind in ("population", "gait"):
        s = {"case": case, "sim": _handle(case, g), "x0": x0, "v0": np.zeros_like(x0), "phase": phase, "amp": amp}
        if kind == "gait":
            s["w"] = np.zeros_like(x0)
            s["w"][:, 0] = g["mass"] / g["mass"].sum()
        return s
    sim = _create(case, g, x0, v0, (0.0, 0.0, 0.0) if kind == "modes" else GRAVITY)
    if g.get("n_groups"):
        CR.cronos_set_actuation(sim, phase, amp, 2.0)
    return {"case": case, "sim": sim, "seed": seed}


FIELDS = ("ke", "pe_spring", "pe_grav", "pe_contact", "mass")
VECTORS = ("p", "com", "bbox_min", "bbox_max")


def _frame(sim):
    x, v, _ = CR.cronos_read_state(sim)
    return {"x": x.astype(np.float32), "v": v.astype(np.float32)}


def _diagnostics(sim):
    diags = CR.cronos_diagnostics(sim)
    out = {f: np.array([d[f] for d in diags], np.float32) for f in FIELDS}
    out.update({f: np.array([d[f] for d in diags], np.float32) for f in VECTORS})
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "frame":
        CR.cronos_step(state["sim"], case["steps"])
        return _frame(state["sim"])
    if kind == "population":
        CR.cronos_set_state(state["sim"], state["x0"], state["v0"], 0)
        CR.cronos_set_actuation(state["sim"], state["phase"], state["amp"], 2.0)
        CR.cronos_step(state["sim"], case["steps"])
        return {"diagnostics": _diagnostics(state["sim"]), **_frame(state["sim"])}
    if kind == "gait":
        CR.cronos_set_state(state["sim"], state["x0"], state["v0"], 0)
        CR.cronos_set_actuation(state["sim"], state["phase"], state["amp"], 2.0)
        loss = CR.cronos_rollout(state["sim"], case["steps"], case["ckpt"], state["w"])
        grads = CR.cronos_rollout_backward(state["sim"], want_state=True)
        return {"loss": np.array([loss], np.float32),
                **{n: a.astype(np.float32) for n, a in zip(("dphase", "damp", "dx0", "dv0"), grads)}}
    if kind == "modes":
        omega, _ = CR.cronos_natural_frequencies(state["sim"], n_modes=case["modes"], tol=1e-10, seed=1 + state["seed"])
        return {"omega": omega}
    if kind == "inspect":
        return {"force": CR.cronos_eval_forces(state["sim"]).astype(np.float32),
                "diagnostics": _diagnostics(state["sim"]), **_frame(state["sim"])}
    if kind == "train":
        loss = CR.cronos_mlp_train(state["net"], state["X"], state["T"], batch=case["batch"], epochs=case["epochs"],
                                   lr=1e-3, seed=4, lr_final=0.0)
        params = CR.cronos_mlp_get_params(state["net"])
        return {"loss": np.array([loss], np.float32), "params": [p.astype(np.float32) for p in params]}
    if kind == "gradient":
        loss, grads = CR.cronos_mlp_loss_grad(state["net"], state["X"], state["T"])
        return {"loss": np.array([loss], np.float32), "grads": [q.astype(np.float32) for q in grads]}
    return {"y": CR.cronos_mlp_forward(state["net"], state["X"])}


# ------------------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: every input and result once, and per step the state in and out (x, v, 1/m: 28 B a
    mass in, 24 B out; one byte-pair per incidence of a body whose springs must be listed).  Flops:
    per step and spring 13 for the length and elongation, 5 for the factor and 12 for the two
    ends' sums; per mass 18."""
    kind = case["kind"]
    if kind in ("train", "screen", "gradient"):
        sizes = (NET_IN,) + (case["width"],) * 3 + (NET_OUT,)
        w = [i * o for i, o in zip(sizes, sizes[1:])]
        n = sum(w) + sum(sizes[1:])
        if kind == "screen":
            return {"bytes": 4 * (n + case["rows"] * (NET_IN + NET_OUT)), "flops": 2.0 * case["rows"] * sum(w)}
        epochs = case.get("epochs", 1)
        batches = epochs * -(-case["rows"] // case.get("batch", case["rows"]))
        # training reads and writes the parameters and both moments each minibatch
        return {"bytes": 4 * ((24 // 4) * n * batches + epochs * case["rows"] * (NET_IN + NET_OUT)),
                "flops": 2.0 * epochs * case["rows"] * (3 * sum(w) - w[0])}
    g = _of(case)
    n, s = len(g["x"]), len(g["k"])
    box = case.get("body") in ("beam", "cube") or kind == "modes"
    entries = 0 if box else 4 * s
    if kind == "modes":
        # one application per Lanczos step; a Krylov space of sqrt(condition) size, at least a hundred
        its = max(100, 4 * case["nx"])
        return {"bytes": its * (16 + 8 + 4 * 24) * n, "flops": its * (60.0 * s + 30.0 * n)}
    if kind == "inspect":
        return {"bytes": (28 + 36) * n, "flops": 50.0 * s + 40.0 * n}
    steps = case["steps"]
    flops = steps * (30.0 * s + 18.0 * n)
    bytes_ = steps * (52 * n + entries) + 48 * n
    if kind == "gait":  # the forward, its recompute and the adjoint (about twice a step's arithmetic)
        return {"bytes": 4 * bytes_, "flops": 4 * flops}
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------------------------ the same in 64 bits

class _Exact:
    """The system's step and energies in FP64, plain torch."""

    def __init__(self, case, g, gravity=GRAVITY, phase=None, amp=None):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        t = lambda a, d=torch.float64: torch.as_tensor(np.asarray(a), dtype=d, device=self.dev)
        self.i, self.j = t(g["ends"][:, 0], torch.int64), t(g["ends"][:, 1], torch.int64)
        self.k, self.rest, self.mass = t(g["k"]), t(g["rest"]), t(g["mass"])[:, None]
        self.g, self.dt, self.damping, self.ground = t(gravity)[None], g["dt"], g["damping"], g["ground"]
        self.free = None if "pinned" not in g else 1.0 - t(g["pinned"])[:, None]
        self.gidx = None
        if g.get("n_groups"):
            body = g["spring_body"] * g["n_groups"]
            count = g["n_groups"] * (len(g["body_offset"]) - 1)
            self.gidx = t(np.where(g["group"] >= 0, body + g["group"], count), torch.int64)
            self.phase, self.amp = t(phase), t(amp)
        self.t = t

    def lengths(self, n, phase=None, amp=None):
        if self.gidx is None:
            return self.rest
        phase, amp = (self.phase, self.amp) if phase is None else (phase, amp)
        a = amp * torch.sin(2.0 * math.pi * 2.0 * n * self.dt + phase)
        return self.rest * (1.0 + torch.cat([a, a.new_zeros(1)])[self.gidx])

    def springs(self, x, l0):
        d = x[self.j] - x[self.i]
        l = d.square().sum(1).sqrt()
        f = (self.k * (l - l0) / l)[:, None] * d
        return torch.zeros_like(x).index_add(0, self.i, f).index_add(0, self.j, -f)

    def normal(self, x):
        return 1.0e5 * torch.clamp(-x[:, 2:], min=0.0)

    def force(self, x, l0):
        f = self.springs(x, l0) + self.mass * self.g
        if self.ground:
            f = f + torch.cat([torch.zeros_like(x[:, :2]), self.normal(x)], 1)
        return f

    def step(self, x, v, n, kick=1.0, phase=None, amp=None):
        h = kick * self.dt
        v = v + h * self.force(x, self.lengths(n, phase, amp)) / self.mass
        if self.ground:
            c = 0.8 * self.normal(x) * h / self.mass
            sq = v[:, :2].square().sum(1, keepdim=True)
            speed = torch.where(sq > 0, sq, torch.ones_like(sq)).sqrt() * (sq > 0)
            keep = torch.where(speed > c, (speed - c) / torch.where(speed > 0, speed, torch.ones_like(speed)),
                               (c <= 0).to(v.dtype))
            v = torch.cat([v[:, :2] * keep, v[:, 2:]], 1)
        v = v * (1.0 - self.damping)
        if self.free is not None:
            v = v * self.free
        return x + self.dt * v, v

    def run(self, x, v, steps, verlet=False):
        for n in range(steps):
            x, v = self.step(x, v, n, 0.5 if verlet and n == 0 else 1.0)
        return x, v

    def diagnostics(self, g, x, v, n):
        offset = g.get("body_offset", np.array([0, len(g["x"])]))
        count = len(offset) - 1
        body = self.t(np.repeat(np.arange(count), np.diff(offset)), torch.int64)
        total = lambda a, at: torch.zeros((count,) + a.shape[1:], dtype=a.dtype, device=a.device).index_add(0, at, a)
        l = (x[self.j] - x[self.i]).square().sum(1).sqrt()
        m = self.mass[:, 0]
        out = {"ke": total(0.5 * m * v.square().sum(1), body),
               "pe_spring": total(0.5 * self.k * (l - self.lengths(n)).square(), body[self.i]),
               "pe_grav": total(-m * (x * self.g).sum(1), body),
               "pe_contact": total(0.5 * 1.0e5 * torch.clamp(-x[:, 2], min=0.0).square() * self.ground, body),
               "mass": total(m, body), "p": total(self.mass * v, body)}
        out["com"] = total(self.mass * x, body) / out["mass"][:, None]
        split = torch.split(x, np.diff(offset).tolist())
        out["bbox_min"] = torch.stack([s.amin(0) for s in split])
        out["bbox_max"] = torch.stack([s.amax(0) for s in split])
        return {f: a.cpu().numpy() for f, a in out.items()}


def _exact_modes(case, g, x0, wanted):
    """Lowest frequencies by Lanczos with full reorthogonalisation on M^-1/2 K M^-1/2."""
    e = _Exact(case, g, (0.0, 0.0, 0.0))
    f32 = lambda a: a.float().double()  # the body as the device holds it
    lift = 1.0  # the device's frame puts the body between one and two units' resolution off zero
    while lift < 8.0 * float(e.rest.max()):
        lift *= 2.0
    while lift > 16.0 * float(e.rest.max()):
        lift *= 0.5
    x = e.t(x0)
    x = f32(x - (x.amin(0, keepdim=True) - lift))
    k, rest = f32(e.k), f32(e.rest)
    d = x[e.j] - x[e.i]
    l = d.square().sum(1, keepdim=True).sqrt()
    nrm, geo = d / l, 1.0 - rest[:, None] / l
    s = e.free / f32(e.mass).sqrt()

    def apply(q):
        u = s * q
        du = u[e.j] - u[e.i]
        along = nrm * (nrm * du).sum(1, keepdim=True)
        f = k[:, None] * (along + geo * (du - along))
        return s * torch.zeros_like(u).index_add(0, e.i, -f).index_add(0, e.j, f)

    n = 3 * len(x0)
    most = min(n, 2500)
    Q = torch.empty((most + 1, n), dtype=torch.float64, device=e.dev)
    gen = torch.Generator().manual_seed(7)
    q = (torch.rand(x0.shape, generator=gen, dtype=torch.float64).to(e.dev) - 0.5) * (e.free > 0)
    Q[0] = (q / q.norm()).ravel()
    a, b, last = [], [], None
    for it in range(most):
        w = apply(Q[it].view(-1, 3)).ravel()
        a.append(float(w @ Q[it]))
        for _ in range(2):
            w = w - Q[:it + 1].T @ (Q[:it + 1] @ w)
        b.append(float(w.norm()))
        Q[it + 1] = w / b[-1]
        if (it + 1) % 100 == 0 or it + 1 == most:
            th, vec = np.linalg.eigh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
            th = th[:wanted]
            if last is not None and np.all(np.abs(th - last) <= 1e-8 * np.abs(th)):
                # the Rayleigh quotients of the Ritz vectors, from the springs' energies: the
                # tridiagonal matrix gives its small eigenvalues to eps of its largest only
                out = []
                for c in range(wanted):
                    y = (Q[:it + 1].T @ e.t(vec[:, c])).view(-1, 3)
                    du = (s * y)[e.j] - (s * y)[e.i]
                    along = (nrm * du).sum(1).square()
                    energy = k * (along + geo[:, 0] * (du.square().sum(1) - along))
                    out.append(float(energy.sum() / y.square().sum()))
                return {"omega": np.sqrt(np.array(out))}
            last = th
    return None


def _exact_network(case, seed):
    sizes, params, X, T = _network(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)
    P = [t(p).requires_grad_(case["kind"] != "screen") for p in params]
    X, T = t(X), t(T)

    def forward(h):
        for l in range(4):
            h = h @ P[2 * l] + P[2 * l + 1]
            h = torch.nn.functional.gelu(h) if l < 3 else h
        return h

    host = lambda a: a.detach().cpu().numpy()
    if case["kind"] == "screen":
        return {"y": host(forward(X))}
    if case["kind"] == "gradient":
        loss = (forward(X) - T).square().mean()
        return {"loss": np.array([float(loss)]), "grads": [host(q) for q in torch.autograd.grad(loss, P)]}
    rows, batch, epochs = case["rows"], case["batch"], case["epochs"]
    mask = (1 << 64) - 1

    def mix(z):  # SplitMix64 (Steele, Lea & Flood 2014), which orders each epoch's rows
        z = (z + 0x9E3779B97F4A7C15) & mask
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        return z ^ (z >> 31)

    M, V = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    step, per = 0, -(-rows // batch)
    total = 0.0
    for e in range(epochs):
        perm = list(range(rows))
        base = mix(4 ^ ((0x5851F42D4C957F2D * (e + 1)) & mask))
        for i in range(rows - 1, 0, -1):
            r = mix(base ^ i) % (i + 1)
            perm[i], perm[r] = perm[r], perm[i]
        perm, total = torch.as_tensor(perm, device=dev), 0.0
        for b in range(0, rows, batch):
            at = perm[b:b + batch]
            loss = (forward(X[at]) - T[at]).square().mean()
            total += float(loss) * len(at)
            grads = torch.autograd.grad(loss, P)
            lr = 0.5 * 1e-3 * (1.0 + math.cos(math.pi * step / max(1, per * epochs - 1)))
            step += 1
            with torch.no_grad():
                for p, q, m, v in zip(P, grads, M, V):
                    m.mul_(0.9).add_(q, alpha=0.1)
                    v.mul_(0.999).addcmul_(q, q, value=0.001)
                    p -= lr * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
    return {"loss": np.array([total / rows]), "params": [host(p) for p in P]}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("train", "screen", "gradient"):
        return _exact_network(case, seed)
    g = _of(case)
    x0, v0, phase, amp = _inputs(g, seed)
    host = lambda a: a.detach().cpu().numpy()
    if kind == "modes":
        return _exact_modes(case, g, x0, case["modes"])
    e = _Exact(case, g, phase=phase, amp=amp)
    if kind == "inspect":
        x, v = e.t(x0), e.t(v0)
        return {"force": host(e.force(x, e.lengths(0))), "diagnostics": e.diagnostics(g, x, v, 0), "x": x0, "v": v0}
    if kind == "gait":
        x, v = e.t(x0).requires_grad_(True), torch.zeros(x0.shape, dtype=torch.float64, device=e.dev, requires_grad=True)
        ph, am = e.phase.requires_grad_(True), e.amp.requires_grad_(True)
        xs, vs = x, v
        for n in range(case["steps"]):
            xs, vs = torch.utils.checkpoint.checkpoint(e.step, xs, vs, n, 1.0, ph, am, use_reentrant=False)
        w = e.mass[:, 0] / e.mass.sum()
        loss = (w * xs[:, 0]).sum()
        dp, da, dx, dv = torch.autograd.grad(loss, (ph, am, x, v))
        return {"loss": np.array([float(loss)]), "dphase": host(dp), "damp": host(da), "dx0": host(dx), "dv0": host(dv)}
    start = np.zeros_like(v0) if kind == "population" else v0
    x, v = e.run(e.t(x0), e.t(start), case["steps"], bool(case.get("verlet")))
    out = {"x": host(x), "v": host(v)}
    if kind == "population":
        out["diagnostics"] = e.diagnostics(g, x, v, case["steps"])
    return out
