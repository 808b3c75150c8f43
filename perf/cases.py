"""The work that users of this framework have it do, as cases that can be timed
and compared: coupled lattice-Boltzmann / metaball steps from the smallest box
to the largest suspension, an ensemble of systems, the read-out of the fluid
fields, the Metaball-Imaging fit (fitness, genetic algorithm, gradient
search), the shape descriptors and the training of the warm-start network.

listed() gives the cases, draw(rng) one more of the same ranges; prepare(case,
seed) what a program holds before the call, run(state) one pass through the
public entry points, work(case) the bytes and operations that a pass cannot do
without, and exact(case, seed) the outputs of the first pass in 64 bits from
the definitions alone.

A step case advances `steps` lattice steps and reads the particles back, as a
program that records a trajectory does; `steps` is even, so that the current
populations are the first of the two buffers in the caller's arena (runs of
1024 nodes, each run holding its 19 populations one after another).
"""
import ctypes as C
import math

import numpy as np
import torch

import paper_2209_10411_amd as mdl
import workloads

DEV = "cuda:0"
RUN = 1024  # nodes per run of the population layout
STORAGE = {"fp32": (workloads.STORE_F32, torch.float32, 4), "fp16": (workloads.STORE_F16, torch.float16, 2),
           "bf16": (workloads.STORE_BF16, torch.bfloat16, 2)}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one body in a small column, periodic in z: a quick look at a single
        # particle, hundreds of thousands of short steps (launches and latency)
        {"name": "step_small", "kind": "step", "nx": 48, "ny": 48, "nz": 80, "zper": True, "storage": "fp32",
         "bodies": 1, "steps": 40},
        # the settling body of the benchmark, 128 x 128 x 384, walls
        {"name": "step_settling", "kind": "step", "nx": 128, "ny": 128, "nz": 384, "zper": False, "storage": "fp32",
         "bodies": 1, "steps": 20},
        # drafting and kissing: two bodies in 160 x 160 x 640, contact on,
        # 16-bit storage (rows that are no multiple of a wave)
        {"name": "step_pair", "kind": "step", "nx": 160, "ny": 160, "nz": 640, "zper": False, "storage": "fp16",
         "bodies": 2, "steps": 10},
        # the 256^3 suspension of 200 bodies, contact on
        {"name": "step_suspension", "kind": "suspension", "box": 256, "bodies": 200, "storage": "fp32", "steps": 10},
        # a parameter sweep: systems of different sizes stepped together
        {"name": "step_ensemble", "kind": "ensemble", "systems": 24, "ragged": False, "storage": "fp32", "steps": 12},
        # writing a snapshot: density and velocity of every node to the host
        {"name": "fields", "kind": "fields", "nx": 96, "ny": 96, "nz": 161, "storage": "fp32"},
        # the fitness of a handful of candidates on a coarse hull
        {"name": "fitness_small", "kind": "fitness", "individuals": 64, "points": 500, "cps": 8},
        # the fitness of one generation at the paper's settings
        {"name": "fitness_large", "kind": "fitness", "individuals": 2400, "points": 4096, "cps": 25},
        # generations of the genetic algorithm at the paper's settings
        {"name": "ga", "kind": "ga", "individuals": 1200, "points": 4096, "cps": 25, "generations": 5},
        # gradient search of a batch of scanned particles
        {"name": "gs", "kind": "gs", "models": 64, "points": 1500, "cps": 25, "steps": 20},
        # sphericity and Corey factor of one body
        {"name": "shape", "kind": "shape", "cps": 8, "radius": 10.0, "cell": 0.2},
        # an epoch of the warm-start network's training
        {"name": "train", "kind": "train", "samples": 8192, "batch": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "suspension", "ensemble", "fields", "fitness", "ga", "gs", "shape",
                       "train"])
    storage = rng.choice(["fp32", "fp32", "fp16", "bf16"])
    if kind == "step":
        nx, ny, nz = _log_int(rng, 40, 160), _log_int(rng, 40, 160), _log_int(rng, 80, 640)
        return {"kind": "step", "nx": nx, "ny": ny, "nz": nz, "zper": rng.random() < 0.4, "storage": storage,
                "bodies": 1 if nz < 3 * min(nx, ny) else rng.choice([1, 2]), "steps": 40 if nx * ny * nz < 1e6 else 10}
    if kind == "suspension":
        box = _log_int(rng, 96, 224)
        return {"kind": "suspension", "box": box, "bodies": max(4, int(200 * (box / 256.0) ** 3)), "storage": storage,
                "steps": 10}
    if kind == "ensemble":
        return {"kind": "ensemble", "systems": rng.randint(3, 20), "ragged": rng.random() < 0.5, "storage": storage,
                "steps": 6 * rng.randint(1, 2)}
    if kind == "fields":
        return {"kind": "fields", "nx": _log_int(rng, 40, 120), "ny": _log_int(rng, 40, 120),
                "nz": _log_int(rng, 48, 120), "storage": storage}
    if kind == "fitness":
        return {"kind": "fitness", "individuals": _log_int(rng, 16, 2400), "points": _log_int(rng, 200, 4096),
                "cps": rng.randint(4, 25)}
    if kind == "ga":
        return {"kind": "ga", "individuals": _log_int(rng, 40, 1200), "points": _log_int(rng, 300, 4096),
                "cps": rng.randint(4, 25), "generations": rng.randint(2, 5)}
    if kind == "gs":
        return {"kind": "gs", "models": _log_int(rng, 1, 256), "points": _log_int(rng, 300, 1500),
                "cps": rng.randint(4, 25), "steps": rng.randint(5, 20)}
    if kind == "shape":
        return {"kind": "shape", "cps": rng.randint(1, 16), "radius": round(rng.uniform(4.0, 10.0), 3),
                "cell": round(rng.uniform(0.2, 0.5), 3)}
    return {"kind": "train", "samples": _log_int(rng, 500, 8192), "batch": _log_int(rng, 64, 1024)}


# -------------------------------------------------------------------- inputs
def _rng(seed, tag):
    return np.random.default_rng([int(seed), tag])


def _quat(rng):
    q = rng.normal(size=4)
    return q / np.linalg.norm(q)


def _step_config(case, seed):
    """Bodies of 4 to 12 control points one above the other near the top of
    the column, their bounding spheres a little into each other, each with a
    small velocity and spin."""
    rng = _rng(seed, 1)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    R = min(10.0, min(nx, ny) / 12.8)
    bodies, z, last = [], None, 0.0
    for _ in range(case["bodies"]):
        off, k = workloads.random_body(rng, int(rng.integers(4, 13)), R)
        off -= off.mean(0)
        p = workloads.Particle(cp_xyz=off, cp_k=k, x=np.zeros(3), quat=_quat(rng), density=1.5,
                               v=rng.normal(0.0, 2e-3, 3), omega=rng.normal(0.0, 2e-3, 3))
        rb = p.bounding_radius()
        z = nz - 6.0 - rb if z is None else z - 0.85 * (last + rb)
        last = rb
        p.x = np.array([nx / 2 + rng.uniform(-0.5, 0.5), ny / 2 + rng.uniform(-0.5, 0.5), z])
        bodies.append(p)
    contact = len(bodies) > 1
    return workloads.Config(nx=nx, ny=ny, nz=nz, periodic=workloads.PERIODIC_Z if case["zper"] else 0, tau=0.6,
                            g_particle=np.array([0.0, 0.0, -2e-5]), counter_force=1 if case["zper"] else 0,
                            quad_h=0.25, storage=STORAGE[case["storage"]][0], particles=bodies,
                            contact_kn=20.0 if contact else 0.0)


def _suspension_config(case, seed):
    cfg = workloads.config5(case["bodies"], case["box"], seed=1000 + int(seed) % 1000003)
    rng = _rng(seed, 2)
    for p in cfg.particles:
        p.v, p.omega = rng.normal(0.0, 2e-3, 3), rng.normal(0.0, 2e-3, 3)
    cfg.quad_h, cfg.storage = 0.5, STORAGE[case["storage"]][0]
    return cfg


def _ensemble_configs(case, seed):
    """The settling ensemble's systems (sizes, tau, density ratio), each with
    a body of its own from the seed."""
    out = []
    for i in range(case["systems"]):
        cfg = workloads.config4_case(i, ragged=case["ragged"])
        p, rng = cfg.particles[0], _rng(seed, 100 + i)
        off, p.cp_k = workloads.random_body(rng, int(rng.integers(4, 17)), 10.0 * min(cfg.nx, cfg.ny) / 128.0)
        p.cp_xyz = off - off.mean(0)
        p.x[2] = max(cfg.nz - p.bounding_radius() - 8.0, cfg.nz / 2)
        p.quat, p.v, p.omega = _quat(rng), rng.normal(0.0, 2e-3, 3), rng.normal(0.0, 2e-3, 3)
        cfg.quad_h, cfg.storage = 0.5, STORAGE[case["storage"]][0]
        out.append(cfg)
    return out


def _fields_input(case, seed):
    """A fluid in motion: populations w_i rho0 plus deviations of a Mach
    number below 0.1, and one body."""
    cfg = _step_config({**case, "bodies": 1, "zper": False}, seed)
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 7 + 3)
    f = torch.rand((19, cfg.n_nodes), generator=g, device=DEV, dtype=torch.float64) * 2e-3 - 1e-3
    return cfg, f + torch.tensor(WD, device=DEV, dtype=torch.float64)[:, None]


def _body_hull(rng, m, n_cp, R):
    """m points on the outer surface of a random metaball (radius by
    bisection along m directions), their mean at the origin, the metaball
    [n][4] and the half-spaces of the points' bounding box cut by the
    directions' support planes."""
    off, k = workloads.random_body(rng, n_cp, 0.5 * R)
    off = 0.5 * (off - off.mean(0))
    k = k * 4.0
    d = rng.normal(size=(m, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    lo, hi = np.zeros(m), np.full(m, 4.0 * R)
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        r2 = ((d[:, None, :] * mid[:, None, None] - off) ** 2).sum(-1)
        inside = (k / r2).sum(-1) >= 1.0
        lo, hi = np.where(inside, mid, lo), np.where(inside, hi, mid)
    H = d * lo[:, None]
    shift = H.mean(0)
    H = H - shift
    nrm = rng.normal(size=(64, 3))
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    planes = np.concatenate([nrm, -(H @ nrm.T).max(0)[:, None]], axis=1)
    return H, planes, np.concatenate([k[:, None], off - shift], axis=1)


def _population(rng, H, P, n):
    r = np.linalg.norm(H, axis=1).mean()
    pop = np.empty((P, n, 4))
    d = rng.normal(size=(P, n, 3))
    pop[..., 1:] = d / np.linalg.norm(d, axis=-1, keepdims=True) * (0.8 * r * rng.random((P, n, 1)) ** (1 / 3))
    pop[..., 0] = rng.uniform(0.02, 2.0, (P, n)) * r * r / n
    return pop


def _dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def _fit_input(case, seed):
    rng = _rng(seed, 3)
    H, _, _ = _body_hull(rng, case["points"], 8, 10.0)
    return rng, H, _population(rng, H, case["individuals"], case["cps"])


def _ga_input(case, seed):
    rng, H, pop = _fit_input(case, seed)
    shape = (case["generations"],) + pop.shape
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 11 + 5)
    U = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    Z = torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)
    perm = np.stack([rng.permutation(pop.shape[0]) for _ in range(case["generations"])]).astype(np.int32)
    return (_dev(H), _dev(pop), U, Z, torch.as_tensor(perm).to(DEV), 0.05 * float(np.abs(H).max()),
            0.2 * float(pop[..., 0].mean()))


def _gs_input(case, seed):
    """Hulls of 60 to 100 % of `points`, each with a start near its metaball."""
    rng = _rng(seed, 4)
    hulls, planes, starts = [], [], []
    for _ in range(case["models"]):
        m = int(rng.integers(int(0.6 * case["points"]), case["points"] + 1))
        H, pl, M = _body_hull(rng, m, case["cps"], 10.0)
        M = M.copy()
        M[:, 1:] += rng.normal(0.0, 0.2, M[:, 1:].shape)
        M[:, 0] *= rng.uniform(0.8, 1.2, len(M))
        hulls.append(H)
        planes.append(pl)
        starts.append(M)
    return hulls, planes, np.stack(starts)


def _shape_input(case, seed):
    rng = _rng(seed, 5)
    return workloads.random_body(rng, case["cps"], case["radius"])


def _train_input(case, seed):
    """Samples of the network's two tasks: a link's node and direction (or a
    partner's centroid), the body's sorted points, and targets."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 13 + 7)
    n = case["samples"]
    x = torch.randn((n, 87), generator=g, device=DEV) * 0.5
    task = (torch.rand(n, generator=g, device=DEV) < 0.2).float()
    x[:, 6] = task
    x[:, 10::4] = torch.rand((n, 20), generator=g, device=DEV) * 0.1
    t = torch.rand((n, 4), generator=g, device=DEV)
    t[:, 0] *= 1.0 - task
    t[:, 1:] *= task[:, None]
    return x.half().contiguous(), t.contiguous(), workloads.mlp_init(int(seed) % 1000003).astype(np.float32)


# ----------------------------------------------------------- prepare and run
def _population_view(arena, offset, n_nodes, storage):
    """The first population buffer of a system's arena as [runs][19][1024];
    the nodes that pad the last run are set to zero once."""
    _, dtype, size = STORAGE[storage]
    runs = -(-n_nodes // RUN)
    v = arena[offset:offset + runs * 19 * RUN * size].view(dtype).view(runs, 19, RUN)
    if n_nodes % RUN:
        v[-1, :, n_nodes % RUN:] = 0
    return v


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "suspension"):
        cfg = _step_config(case, seed) if kind == "step" else _suspension_config(case, seed)
        sim = mdl.Simulation(cfg, device=DEV)
        return {"kind": "step", "sim": sim, "steps": case["steps"],
                "pop": _population_view(sim.arena, 0, cfg.n_nodes, case["storage"])}
    if kind == "ensemble":
        cfgs = _ensemble_configs(case, seed)
        ens = mdl.Ensemble(cfgs, device=DEV)
        ens.autotune(budget_ms=300.0)
        offset, pops = 0, []
        for cfg in cfgs:
            pops.append(_population_view(ens.arena, offset, cfg.n_nodes, case["storage"]))
            offset += mdl.arena_bytes(cfg)
        return {"kind": "ensemble", "ens": ens, "steps": case["steps"], "pops": pops}
    if kind == "fields":
        cfg, f = _fields_input(case, seed)
        sim = mdl.Simulation(cfg, device=DEV)
        sim.set_populations(f.cpu().numpy(), post_collision=True)
        return {"kind": "fields", "sim": sim}
    if kind == "fitness":
        _, H, pop = _fit_input(case, seed)
        P, m = case["individuals"], case["points"]
        wb = int(mdl.lib().mi_fitness_work_bytes(m, P))
        return {"kind": "fitness", "H": _dev(H), "pop": _dev(pop), "n": case["cps"],
                "F": torch.empty(P, dtype=torch.float64, device=DEV),
                "work": torch.empty(max(wb, 1), dtype=torch.uint8, device=DEV), "wb": wb}
    if kind == "ga":
        H, pop, U, Z, perm, sx, sk = _ga_input(case, seed)
        N, n = case["individuals"], case["cps"]
        wb = int(mdl.lib().mi_ga_work_bytes(case["points"], N, n))
        return {"kind": "ga", "H": H, "pop0": pop, "pop": torch.empty_like(pop), "U": U, "Z": Z, "perm": perm,
                "sx": sx, "sk": sk, "E": case["generations"],
                "F": torch.empty(N, dtype=torch.float64, device=DEV),
                "work": torch.empty(wb, dtype=torch.uint8, device=DEV), "wb": wb}
    if kind == "gs":
        hulls, planes, M0 = _gs_input(case, seed)
        off = lambda xs: _dev(np.concatenate([[0], np.cumsum([len(x) for x in xs])]), torch.int64)  # noqa: E731
        M0 = _dev(M0)
        return {"kind": "gs", "H": _dev(np.concatenate(hulls)), "ho": off(hulls), "pl": _dev(np.concatenate(planes)),
                "po": off(planes), "M0": M0, "M": torch.empty_like(M0), "E": case["steps"],
                "loss": torch.empty((case["models"], 3), dtype=torch.float64, device=DEV)}
    if kind == "shape":
        cp, k = _shape_input(case, seed)
        return {"kind": "shape", "cp": cp, "k": k, "h": case["cell"]}
    x, t, params = _train_input(case, seed)
    return {"kind": "train", "net": mdl.Mlp(params, device=DEV), "x": x, "t": t, "batch": case["batch"]}


def _ptr(t):
    return C.c_void_p(t.data_ptr())


def _checked(rc):
    if rc != 0:
        raise RuntimeError(f"status {rc}")


def _bodies(sims):
    """The particles' states of every system, stacked as a trajectory holds them."""
    ps = [p for s in sims for p in s.particles()]
    return {key: np.stack([p[key] for p in ps]) for key in ("x", "quat", "v", "omega", "F", "T")}


def run(state):
    kind, L = state["kind"], mdl.lib()
    if kind == "step":
        state["sim"].step(state["steps"])
        return {"populations": state["pop"], "bodies": _bodies([state["sim"]])}
    if kind == "ensemble":
        state["ens"].step(state["steps"])
        return {"populations": state["pops"], "bodies": _bodies(state["ens"].cases)}
    if kind == "fields":
        rho, u = state["sim"].macros()
        return {"rho": rho, "u": u}
    if kind == "shape":
        return mdl.shape_descriptors(state["cp"], state["k"], state["h"], device=DEV)
    if kind == "train":
        state["net"].train(state["x"], state["t"], batch=state["batch"], lr=1e-3)
        return {"params": state["net"].params()}
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    if kind == "fitness":
        P, m = state["pop"].shape[0], state["H"].shape[0]
        _checked(L.mi_fitness(_ptr(state["H"]), m, _ptr(state["pop"]), P, state["n"], _ptr(state["F"]),
                              _ptr(state["work"]), state["wb"], stream))
        return {"F": state["F"]}
    if kind == "ga":
        state["pop"].copy_(state["pop0"])
        N, n = state["pop"].shape[:2]
        _checked(L.mi_ga(_ptr(state["H"]), state["H"].shape[0], N, n, state["E"], 0.6, 0.5, state["sx"], state["sk"],
                         _ptr(state["U"]), _ptr(state["Z"]), _ptr(state["perm"]), _ptr(state["pop"]),
                         _ptr(state["F"]), _ptr(state["work"]), state["wb"], stream))
        return {"population": state["pop"], "F": state["F"]}
    state["M"].copy_(state["M0"])
    B, n = state["M"].shape[:2]
    _checked(L.mi_gs(_ptr(state["H"]), _ptr(state["ho"]), _ptr(state["pl"]), _ptr(state["po"]), B, n, state["E"], 1e-4,
                     _ptr(state["M"]), _ptr(state["loss"]), stream))
    return {"M": state["M"], "loss": state["loss"]}


def work(case):
    """Bytes: every input read once and every output written once (a lattice
    step reads and writes the 19 populations of a node and reads its class
    byte).  Operations of the definitions: 250 per collided node; 10 per
    (hull point, control point) of f, 14 more of its gradient; 8 per (grid
    sample, control point); 6 per parameter and sample of the network."""
    kind = case["kind"]
    if kind in ("step", "suspension", "ensemble"):
        size = STORAGE[case["storage"]][2]
        if kind == "step":
            N = case["nx"] * case["ny"] * case["nz"]
        elif kind == "suspension":
            N = case["box"] ** 3
        else:
            N = sum(c.n_nodes for c in _ensemble_configs(case, 0))
        return {"bytes": case["steps"] * N * (38 * size + 1), "flops": case["steps"] * N * 250}
    if kind == "fields":
        N = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": N * (19 * STORAGE[case["storage"]][2] + 32), "flops": N * 60}
    if kind == "fitness":
        P, m, n = case["individuals"], case["points"], case["cps"]
        return {"bytes": 24 * m + 32 * P * n + 8 * P, "flops": P * m * (10 * n + 3)}
    if kind == "ga":
        P, m, n, E = case["individuals"], case["points"], case["cps"], case["generations"]
        return {"bytes": 24 * m + E * P * (64 * n + 4) + 2 * P * 32 * n, "flops": (2 * E + 1) * P * m * (10 * n + 3)}
    if kind == "gs":
        B, m, n = case["models"], int(0.8 * case["points"]), case["cps"]
        return {"bytes": B * (24 * m + 64 * n), "flops": B * m * n * (2 * case["steps"] * 24 + 30)}
    if kind == "shape":
        side = 5.0 * case["radius"] / case["cell"]
        return {"bytes": 32 * case["cps"] + 200, "flops": 2 * side ** 3 * 8 * case["cps"]}
    n = case["samples"]
    return {"bytes": n * (87 * 2 + 16) + 3 * 8 * 10052 * -(-n // case["batch"]), "flops": 6 * 10052 * n}


# ------------------------------------------------ the definitions in 64 bits
E3 = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
               (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1),
               (0, 1, -1), (0, -1, 1)])
WD = np.where((E3 ** 2).sum(1) == 0, 1 / 3, np.where((E3 ** 2).sum(1) == 1, 1 / 18, 1 / 36))
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _rotation(q):
    w, x, y, z = q
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                     [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                     [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]])


def _value(x, cp, k, image):
    """sum k / |x - p|^2 at the points x [n][3]."""
    out = torch.zeros(len(x), dtype=torch.float64, device=x.device)
    for p, kk in zip(cp, k):
        d = image(x - torch.tensor(p, dtype=torch.float64, device=x.device))
        out += float(kk) / (d * d).sum(-1)
    return out


class _Body:
    """Volume, centroid and inertia by midpoint cells; pose and motion."""

    def __init__(self, p, h):
        rs = math.sqrt(p.cp_k.sum())
        lo, hi = p.cp_xyz.min(0) - rs, p.cp_xyz.max(0) + rs
        n = np.ceil((hi - lo) / h).astype(int)
        lo = 0.5 * (lo + hi) - 0.5 * n * h
        ax = [torch.tensor(lo[a] + (np.arange(n[a]) + 0.5) * h, device=DEV) for a in range(3)]
        g = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
        pts = g[_value(g, p.cp_xyz, p.cp_k, lambda d: d) >= 1.0]
        c = pts.mean(0)
        r = pts - c
        S = (r.T @ r).cpu().numpy() * h ** 3
        self.V = len(pts) * h ** 3
        self.m = p.density * self.V
        self.I = p.density * (np.trace(S) * np.eye(3) - S)
        self.q = p.quat / np.linalg.norm(p.quat)
        c = c.cpu().numpy()
        self.cpb, self.k = p.cp_xyz - c, p.cp_k
        self.X = p.x + _rotation(self.q) @ c
        self.v, self.w = np.array(p.v, float), np.array(p.omega, float)
        self.F, self.T = np.zeros(3), np.zeros(3)

    def points(self):
        return self.X + self.cpb @ _rotation(self.q).T

    def advance(self, weight, L, periodic):
        self.v = self.v + (self.F + weight) / self.m
        self.X = self.X + self.v
        R = _rotation(self.q)
        wb = R.T @ self.w
        wb = wb + np.linalg.solve(self.I, R.T @ self.T - np.cross(wb, self.I @ wb))
        self.w = R @ wb
        a = np.linalg.norm(wb)
        dq = np.concatenate([[math.cos(0.5 * a)], wb * (math.sin(0.5 * a) / a if a else 0.5)])
        a0, b0 = self.q[0], self.q[1:]
        q = np.concatenate([[a0 * dq[0] - b0 @ dq[1:]], a0 * dq[1:] + dq[0] * b0 + np.cross(b0, dq[1:])])
        self.q = q / np.linalg.norm(q)
        for c in range(3):
            if periodic >> c & 1:
                self.X[c] -= L[c] * math.floor(self.X[c] / L[c])


class _Exact:
    """The coupled step without body contacts: deviations d [19][N], x fastest."""

    def __init__(self, cfg):
        self.cfg, self.L = cfg, np.array([cfg.nx, cfg.ny, cfg.nz])
        N = cfg.n_nodes
        n = torch.arange(N, device=DEV)
        self.xyz = torch.stack([n % cfg.nx, n // cfg.nx % cfg.ny, n // (cfg.nx * cfg.ny)], -1)
        self.bodies = [_Body(p, cfg.quad_h) for p in cfg.particles]
        self.E = torch.tensor(E3, dtype=torch.float64, device=DEV)
        self.W = torch.tensor(WD, device=DEV)
        self.opp = torch.tensor(OPP, device=DEV)
        self.neighbour = [self.source(n, self.E[i]) for i in range(19)]
        self.flag()
        self.weight = [(b.m - cfg.rho0 * b.V) * np.asarray(cfg.g_particle, float) for b in self.bodies]
        g = np.array(cfg.g_fluid, float)
        if cfg.counter_force:
            g = g - sum(self.weight) / (cfg.rho0 * float((self.own < 0).sum()))
        self.g = torch.tensor(g, device=DEV)
        self.A = torch.zeros((19, N), dtype=torch.float64, device=DEV)
        self.A = torch.where(self.own < 0, self.collide(self.A), self.A)
        self.B = torch.zeros_like(self.A)

    def image(self, d):
        d = d.clone()
        for a in range(3):
            if self.cfg.periodic >> a & 1:
                d[..., a] -= self.L[a] * torch.floor(d[..., a] / self.L[a] + 0.5)
        return d

    def flag(self):
        self.own = torch.full((self.cfg.n_nodes,), -1, device=DEV)
        for b in reversed(range(len(self.bodies))):
            body = self.bodies[b]
            near = (self.image(self.xyz - torch.tensor(body.X, device=DEV)).abs() <
                    np.abs(body.cpb).max() * 2 + math.sqrt(body.k.sum())).all(-1).nonzero()[:, 0]
            C = _value(self.xyz[near].double(), body.points(), body.k, self.image)
            self.own[near[C >= 1.0]] = b

    def source(self, node, e, sign=-1):
        """The nodes x + sign e (e [3] or [n][3]) and whether they lie in the domain."""
        c = self.xyz[node] + sign * e.long()
        ok = torch.ones(len(node), dtype=torch.bool, device=DEV)
        for a in range(3):
            if not self.cfg.periodic >> a & 1:
                ok &= (c[:, a] >= 0) & (c[:, a] < int(self.L[a]))
            c[:, a] %= int(self.L[a])
        return c[:, 0] + self.cfg.nx * (c[:, 1] + self.cfg.ny * c[:, 2]), ok

    def feq(self, rho, u, i):
        """Equilibrium of direction i (one, or one per row of u)."""
        eu = (u * self.E[i]).sum(-1)
        return self.W[i] * rho * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * (u * u).sum(-1))

    def collide(self, d):
        rho = self.cfg.rho0 + d.sum(0)
        F = rho[:, None] * self.g
        u = (torch.stack([(self.E[:, a, None] * d).sum(0) for a in range(3)], -1) + 0.5 * F) / rho[:, None]
        om = 1.0 / self.cfg.tau
        out = torch.empty_like(d)
        uF = (u * F).sum(-1)
        for i in range(19):
            eF, eu = F @ self.E[i], u @ self.E[i]
            src = WD[i] * (1 - 0.5 * om) * (3 * (eF - uF) + 9 * eu * eF)
            out[i] = d[i] + om * (self.feq(rho, u, i) - WD[i] * self.cfg.rho0 - d[i]) + src
        return out

    def moments(self, node):
        d = self.A[:, node]
        rho = self.cfg.rho0 + d.sum(0)
        return rho, (self.E.T @ d).T / rho[:, None] - 0.5 * self.g

    def fraction(self, node, e, body):
        cp, k = torch.tensor(body.points(), device=DEV), torch.tensor(body.k, device=DEV)
        x = self.xyz[node].double()

        def inside(s):
            d = self.image((x - s[:, None] * e)[:, None] - cp)
            return (k / (d * d).sum(-1)).sum(-1) >= 1.0

        hi = torch.ones(len(node), dtype=torch.float64, device=DEV)
        for j in range(7, 0, -1):
            s = torch.full_like(hi, j / 8)
            hi = torch.where(inside(s), s, hi)
        lo = hi - 0.125
        for _ in range(50):
            mid = 0.5 * (lo + hi)
            into = inside(mid)
            lo, hi = torch.where(into, lo, mid), torch.where(into, mid, hi)
        return 0.5 * (lo + hi)

    def bounce(self, node, i, b):
        """Incoming deviations on the links (node [n], direction i [n]) cut by
        body b; their momentum exchange becomes the body's load."""
        body, rho0 = self.bodies[b], self.cfg.rho0
        ib, w, e = self.opp[i], self.W[i], self.E[i]
        ff, ok = self.source(node, e, +1)
        ibb = ok & (self.own[ff] < 0) if self.cfg.bc == 1 else torch.zeros_like(ok)
        q = torch.where(ibb, self.fraction(node, e, body), torch.full_like(w, 0.5))[:, None]
        r = self.image(self.xyz[node] - q * e - torch.tensor(body.X, device=DEV))
        uw = torch.tensor(body.v, device=DEV) + torch.linalg.cross(torch.tensor(body.w, device=DEV).expand_as(r), r)
        fb = self.A[ib, node]
        mw = 6 * w * rho0 * (uw * e).sum(-1)
        rho, uf = self.moments(node)
        _, uff = self.moments(ff)
        us = torch.where(q <= 0.5, 2 * q * uf + (1 - 2 * q) * uff, (1 - q) / q * uf + (2 * q - 1) / q * uw)
        ud = us / 3 + 2 / 3 * ((1 - q) / (1 + q) * uff + 2 * q / (1 + q) * uw)
        val = fb + mw + torch.where(ibb, self.feq(rho, ud, ib) - self.feq(rho, uf, ib), torch.zeros_like(fb))
        dP = (-e - uw) * fb[:, None] - (e - uw) * val[:, None]
        body.F, body.T = dP.sum(0).cpu().numpy(), torch.linalg.cross(r, dP).sum(0).cpu().numpy()
        return val

    def step(self):
        old, d = self.own, torch.empty_like(self.A)
        d[0] = self.A[0]
        usable = torch.ones_like(d, dtype=torch.bool)  # came from a fluid node
        usable[0] = old < 0
        links = []
        for i in range(1, 19):
            src, ok = self.neighbour[i]
            d[i] = torch.where(ok, self.A[i, src], self.A[OPP[i]])
            behind = torch.where(ok, old[src], torch.full_like(old, -1))
            usable[i] = ok & (behind < 0)
            node = ((behind >= 0) & (old < 0)).nonzero()[:, 0]
            links.append(torch.stack([node, torch.full_like(node, i), behind[node]]))
        links = torch.cat(links, 1)
        for b in range(len(self.bodies)):
            node, i, _ = links[:, links[2] == b]
            # the value also stays in the destination of a node that is covered now
            d[i, node] = self.B[i, node] = self.bounce(node, i, b)
        for body, weight in zip(self.bodies, self.weight):
            body.advance(weight, self.L, self.cfg.periodic)
        self.flag()
        new = ((old >= 0) & (self.own < 0)).nonzero()[:, 0]
        if len(new):
            X, V, Om = (torch.tensor(np.stack([getattr(b, a) for b in self.bodies]), device=DEV)[old[new]] for a in "Xvw")
            u = V + torch.linalg.cross(Om, self.image(self.xyz[new] - X))
            got, use = d[:, new].clone(), usable[:, new]
            for i in range(19):
                eq = self.feq(torch.full((len(new),), self.cfg.rho0, dtype=torch.float64, device=DEV), u, i)
                fill = torch.where(use[OPP[i]], got[OPP[i]] + 6 * WD[i] * self.cfg.rho0 * (u @ self.E[i]),
                                   eq - WD[i] * self.cfg.rho0)
                d[i, new] = torch.where(use[i], got[i], fill)
        # a solid node keeps what its buffer held
        self.A, self.B = torch.where(self.own < 0, self.collide(d), self.B), self.A

    def populations(self, storage):
        N = self.cfg.n_nodes
        d = torch.zeros((19, -(-N // RUN) * RUN), dtype=torch.float64, device=DEV)
        d[:, :N] = self.A * (1024.0 if storage == "fp16" else 1.0)
        return d.view(19, -1, RUN).permute(1, 0, 2).contiguous()

    def state(self):
        return [{"x": b.X, "quat": b.q, "v": b.v, "omega": b.w, "F": b.F, "T": b.T} for b in self.bodies]


def _exact_steps(cfgs, case):
    pops, ps = [], []
    for cfg in cfgs:
        e = _Exact(cfg)
        for _ in range(case["steps"]):
            e.step()
        pops.append(e.populations(case["storage"]))
        ps += e.state()
    return pops, {key: np.stack([p[key] for p in ps]) for key in ps[0]}


def _exact_fitness(H, pop):
    F = torch.empty(len(pop), dtype=torch.float64, device=DEV)
    for a in range(0, len(pop), 64):
        f = torch.zeros((len(pop[a:a + 64]), len(H)), dtype=torch.float64, device=DEV)
        for j in range(pop.shape[1]):
            d = H[None] - pop[a:a + 64, j, None, 1:]
            f += pop[a:a + 64, j, None, 0] / (d * d).sum(-1)
        F[a:a + 64] = ((f - 1.0) ** 2).sum(1)
    return F


def _exact_ga(case, seed):
    H, pop, U, Z, perm, sx, sk = _ga_input(case, seed)
    N, n, _ = pop.shape
    sigma = torch.tensor([sk, sx, sx, sx], dtype=torch.float64, device=DEV)
    c = int(0.5 * n + 0.5)
    F = _exact_fitness(H, pop)
    for e in range(case["generations"]):
        mutant = pop + torch.where(U[e] < 0.6, Z[e] * sigma, torch.zeros_like(pop))
        mutant[..., 0] = mutant[..., 0].clamp(min=0.0)
        p = perm[e].long()
        kids = pop[p]
        pairs = N // 2 * 2
        other = pop[p[:pairs].view(-1, 2).flip(1).reshape(-1)]
        kids[:pairs, c:] = other[:, c:]
        pool = torch.cat([pop, mutant, kids])
        F = torch.cat([F, _exact_fitness(H, pool[N:])])
        keep = torch.sort(F, stable=True).indices[:N]
        pop, F = pool[keep], F[keep]
    return {"population": pop, "F": F}


def _exact_gs(case, seed):
    hulls, planes, M0 = _gs_input(case, seed)
    B, m = len(hulls), max(len(h) for h in hulls)
    H = torch.zeros((B, m, 3), dtype=torch.float64, device=DEV)
    on = torch.zeros((B, m), dtype=torch.float64, device=DEV)
    for b, h in enumerate(hulls):
        H[b, :len(h)], on[b, :len(h)] = _dev(h), 1.0
    M, pl = _dev(M0), _dev(np.stack(planes))

    def pieces(M):
        d = H[:, :, None] - M[:, None, :, 1:]
        y = 1.0 / (d * d).sum(-1)
        return d, y, (M[:, None, :, 0] * y).sum(-1)

    def loss(M):
        _, _, f = pieces(M)
        low = (f - 1) ** 2 + 1.0 / f.clamp(min=1e-12) - 1.0
        return (on * torch.where(f >= 2, (f - 1) ** 2, torch.where(f >= 1, f - 1, low))).sum(1)

    def descend(M):
        for _ in range(case["steps"]):
            d, y, f = pieces(M)
            low = 2 * (f - 1) - torch.where(f > 1e-12, 1.0 / (f * f), torch.zeros_like(f))
            g = on * torch.where(f >= 2, 2 * (f - 1), torch.where(f >= 1, torch.ones_like(f), low))
            gk = (g[..., None] * y).sum(1)
            gp = ((2 * g[..., None] * M[:, None, :, 0] * y * y)[..., None] * d).sum(1)
            M = M - 1e-4 * torch.cat([gk[..., None], gp], -1)
        return M

    L0 = loss(M)
    M = descend(M)
    L1 = loss(M)
    side = (M[:, :, None, 1:] * pl[:, None, :, :3]).sum(-1) + pl[:, None, :, 3]
    bad = (M[..., 0] < 0) | (side > 0).any(-1)
    M[..., 0] = torch.where(bad, torch.zeros_like(M[..., 0]), M[..., 0])
    M = descend(M)
    return {"M": M, "loss": torch.stack([L0, L1, loss(M)], -1)}


def _exact_shape(case, seed):
    cp, k = _shape_input(case, seed)
    h, r = case["cell"], math.sqrt(k.sum())
    lo = cp.min(0) - r - h
    n = np.ceil((cp.max(0) + r + h - lo) / h).astype(int) + 1
    axes = [torch.arange(int(c), dtype=torch.float64, device=DEV) for c in n]

    def grid(shift):
        return torch.stack(torch.meshgrid(*[lo[a] + h * (axes[a] + shift) for a in range(3)], indexing="ij"), -1)

    same = lambda d: d  # noqa: E731
    centres = grid(0.5).reshape(-1, 3)
    pts = centres[_value(centres, cp, k, same) >= 1.0]
    c = pts.mean(0)
    rel = pts - c
    _, vec = np.linalg.eigh((rel.T @ rel).cpu().numpy())
    vec = vec * np.where(vec[np.abs(vec).argmax(0), range(3)] < 0, -1.0, 1.0)
    pr = rel @ torch.tensor(vec, device=DEV)
    ext = (pr.max(0).values - pr.min(0).values).cpu().numpy()
    order = np.argsort(ext, kind="stable")
    dims, ax = ext[order] + h, vec[:, order]
    # surface: six tetrahedra of every cell between eight grid nodes
    nodes = grid(0.0)
    g = (_value(nodes.reshape(-1, 3), cp, k, same) - 1.0).view(*nodes.shape[:3])
    corner = lambda t, q: t[q & 1:t.shape[0] - 1 + (q & 1), q >> 1 & 1:t.shape[1] - 1 + (q >> 1 & 1),  # noqa: E731
                            q >> 2:t.shape[2] - 1 + (q >> 2)]
    G = torch.stack([corner(g, q).reshape(-1) for q in range(8)], -1)
    mixed = (G.min(1).values < 0) & (G.max(1).values >= 0)
    G = G[mixed]
    P = torch.stack([corner(nodes, q).reshape(-1, 3)[mixed] for q in range(8)], 1)
    area = 0.0
    tri = lambda a, b, d: 0.5 * torch.linalg.norm(torch.linalg.cross(b - a, d - a), dim=-1)  # noqa: E731
    for tet in ((0, 1, 3, 7), (0, 3, 2, 7), (0, 2, 6, 7), (0, 6, 4, 7), (0, 4, 5, 7), (0, 5, 1, 7)):
        gt, pt = G[:, tet], P[:, tet]
        sign = gt >= 0
        count = sign.sum(1)
        for lone, which in ((1, True), (3, False)):
            at = (count == lone).nonzero()[:, 0]
            first = (sign[at] == which).int().argmax(1)
            others = torch.stack([(first + s) % 4 for s in (1, 2, 3)], 1)
            ga, pa = gt[at].gather(1, first[:, None]), pt[at][torch.arange(len(at)), first]
            go = gt[at].gather(1, others)
            po = pt[at].gather(1, others[..., None].expand(-1, -1, 3))
            cut = pa[:, None] + (ga / (ga - go))[..., None] * (po - pa[:, None])
            area += float(tri(cut[:, 0], cut[:, 1], cut[:, 2]).sum())
        at = (count == 2).nonzero()[:, 0]
        idx = torch.argsort(sign[at].int(), dim=1, descending=True, stable=True)
        ga, pa = gt[at].gather(1, idx), pt[at].gather(1, idx[..., None].expand(-1, -1, 3))
        cut = lambda a, b: pa[:, a] + (ga[:, a] / (ga[:, a] - ga[:, b]))[:, None] * (pa[:, b] - pa[:, a])  # noqa: E731
        q0, q1, q2, q3 = cut(0, 2), cut(0, 3), cut(1, 3), cut(1, 2)
        area += float((tri(q0, q1, q2) + tri(q0, q2, q3)).sum())
    # projection along the shortest axis
    half = 0.5 * dims + 2.0 * h
    cnt = np.ceil(2.0 * half / h).astype(int) + 1
    s = [torch.tensor(-half[a] + h * np.arange(cnt[a]), device=DEV) for a in range(3)]
    axd = torch.tensor(ax, device=DEV)
    hit = torch.zeros((int(cnt[2]), int(cnt[1])), dtype=torch.bool, device=DEV)
    plane = c + s[2][:, None, None] * axd[:, 2] + s[1][None, :, None] * axd[:, 1]
    for w in s[0]:
        hit |= (_value((plane + w * axd[:, 0]).reshape(-1, 3), cp, k, same) >= 1.0).view_as(hit)
    hits = int(hit.sum())
    V, Ap = len(pts) * h ** 3, hits * h * h
    d_n = (6.0 * V / math.pi) ** (1 / 3)
    return {"V": V, "S": area, "A_p": Ap, "dims": dims, "axes": ax, "centroid": c.cpu().numpy(), "d_n": d_n,
            "d_s": math.sqrt(4.0 * Ap / math.pi), "Phi": math.pi * d_n * d_n / area,
            "CSF": float(dims[0] / math.sqrt(dims[1] * dims[2])), "cells_inside": len(pts), "columns_hit": hits}


def _exact_train(case, seed):
    x, t, params = _train_input(case, seed)
    x, t = x.double(), t.double()
    p = torch.tensor(params, dtype=torch.float64, device=DEV)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    step = 0
    for a in range(0, case["samples"], case["batch"]):
        xb, tb = x[a:a + case["batch"]], t[a:a + case["batch"]]
        W1, b1, W2, b2, W3, b3 = torch.split(p, [87 * 64, 64, 64 * 64, 64, 64 * 4, 4])
        W1, W2, W3 = W1.view(87, 64), W2.view(64, 64), W3.view(64, 4)
        h1 = torch.tanh(xb @ W1 + b1)
        h2 = torch.tanh(h1 @ W2 + b2)
        on = torch.cat([1.0 - xb[:, 6:7], xb[:, 6:7].expand(-1, 3)], 1)
        dz = 2.0 * on * (h2 @ W3 + b3 - tb) / len(xb)
        dz2 = (dz @ W3.T) * (1 - h2 * h2)
        dz1 = (dz2 @ W2.T) * (1 - h1 * h1)
        g = torch.cat([u.reshape(-1) for u in (xb.T @ dz1, dz1.sum(0), h1.T @ dz2, dz2.sum(0), h2.T @ dz, dz.sum(0))])
        step += 1
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1 - 0.9 ** step)) / (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
    return {"params": p}


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        pops, bodies = _exact_steps([_step_config(case, seed)], case)
        return {"populations": pops[0], "bodies": bodies}
    if kind == "suspension":
        return None  # contacts of hundreds of bodies: minutes in plain torch
    if kind == "ensemble":
        pops, bodies = _exact_steps(_ensemble_configs(case, seed), case)
        return {"populations": pops, "bodies": bodies}
    if kind == "fields":
        cfg, f = _fields_input(case, seed)
        rho = f.sum(0)
        u = (torch.tensor(E3, dtype=torch.float64, device=DEV).T @ f).T / rho[:, None]
        return {"rho": rho.cpu().numpy(), "u": u.cpu().numpy()}
    if kind == "fitness":
        _, H, pop = _fit_input(case, seed)
        return {"F": _exact_fitness(_dev(H), _dev(pop))}
    if kind == "ga":
        return _exact_ga(case, seed)
    if kind == "gs":
        return _exact_gs(case, seed)
    if kind == "shape":
        return _exact_shape(case, seed)
    return _exact_train(case, seed)
