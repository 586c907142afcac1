"""Workloads of the cavity solver that its speed is measured on.

Every case goes through the package's public entry points (Solver, Adjoint, probe_objective,
Pool) as a program of its users does. The kinds:

  evolve     a resident cavity advanced by n steps, its six fields then written into torch
             tensors on the GPU (fdtd_step + fdtd_get_fields_device): every simulation
  roundtrip  NumPy fields in, n steps, NumPy fields out (the README's example)
  monitor    a few steps, then the diagnostics (energy, div B, ...), again and again
  adjoint    J and dJ/d eps_r with a kept Adjoint handle (repeated gradients of one medium)
  objective  probe_objective(eps).backward(): one iteration of a permittivity inversion, where
             eps_r is new in every iteration, so the solver is made anew as well
  pool       a burst of cavity solves through the serving pool, every result fetched

exact() is the same recurrence in FP64 torch on the same inputs, with coefficients that are not
rounded to the storage type.
"""

import math
import random

import numpy as np
import torch

import paper_2504_09118_amd as P
from paper_2504_09118_amd.adjoint import Adjoint, probe_objective

COURANT = 0.5 / math.sqrt(3.0)
DEV = "cuda:0"


def listed():
    return [
        # the paper's smallest cavity, run for a few steps at a time: launches and latency
        {"name": "evolve_16", "kind": "evolve", "nx": 16, "ny": 16, "nz": 16, "steps": 20, "medium": "vacuum",
         "storage": "f32", "dy": 0.0, "dz": 0.0},
        # the README's program on a small per-cell medium: host arrays in and out
        {"name": "roundtrip_64", "kind": "roundtrip", "nx": 64, "ny": 64, "nz": 64, "steps": 100,
         "medium": "spheres", "storage": "f32", "dy": 0.0, "dz": 0.0},
        # an odd cavity with both material arrays, watched while it runs (the parity tests' grid)
        {"name": "monitor_133x40x71", "kind": "monitor", "nx": 133, "ny": 40, "nz": 71, "steps": 5, "reads": 8,
         "medium": "both", "storage": "f32", "dy": 0.0, "dz": 0.0},
        # the middle of the paper's range of sizes
        {"name": "evolve_128", "kind": "evolve", "nx": 128, "ny": 128, "nz": 128, "steps": 200,
         "medium": "spheres", "storage": "f32", "dy": 0.0, "dz": 0.0},
        # rectangular cells: per-node coefficient arrays of both kinds
        {"name": "rect_160x96x128", "kind": "evolve", "nx": 160, "ny": 96, "nz": 128, "steps": 120,
         "medium": "spheres", "storage": "f32", "dy": 0.7, "dz": 1.3},
        # the 256^3 cavity of the schedule table: eps_r and mu_r given as arrays
        {"name": "evolve_256_ce_ch", "kind": "evolve", "nx": 256, "ny": 256, "nz": 256, "steps": 120,
         "medium": "both", "storage": "f32", "dy": 0.0, "dz": 0.0},
        # 16-bit field storage on a large ragged cavity
        {"name": "evolve_f16_394x301x350", "kind": "evolve", "nx": 394, "ny": 301, "nz": 350, "steps": 60,
         "medium": "spheres", "storage": "f16", "dy": 0.0, "dz": 0.0},
        # compensated 16-bit storage
        {"name": "evolve_bf16c_320", "kind": "evolve", "nx": 320, "ny": 320, "nz": 320, "steps": 60,
         "medium": "spheres", "storage": "bf16c", "dy": 0.0, "dz": 0.0},
        # the headline benchmark's cavity: the largest pass
        {"name": "evolve_512", "kind": "evolve", "nx": 512, "ny": 512, "nz": 512, "steps": 100,
         "medium": "spheres", "storage": "f32", "dy": 0.0, "dz": 0.0},
        # the adjoint benchmark's medium with a kept handle: forward and backward
        {"name": "adjoint_128", "kind": "adjoint", "nx": 128, "ny": 128, "nz": 128, "steps": 200, "probes": 8,
         "medium": "random"},
        # one iteration of an inversion on a small grid, through autograd
        {"name": "objective_48x40x56", "kind": "objective", "nx": 48, "ny": 40, "nz": 56, "steps": 150, "probes": 8,
         "medium": "random"},
        # a burst of the serving stream's cavities (its smaller half), results kept and fetched
        {"name": "pool_burst", "kind": "pool", "requests": 10, "lo": 48, "hi": 192, "mix": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve", "evolve", "evolve", "evolve", "roundtrip", "monitor", "adjoint", "objective", "pool"])
    if kind == "pool":
        lo = rng.choice([48, 64])
        return {"kind": kind, "requests": rng.randint(2, 10), "lo": lo, "hi": rng.choice([96, 128, 160, 192]),
                "mix": rng.randint(1, 10 ** 6)}
    top = {"evolve": 480, "roundtrip": 160, "monitor": 224, "adjoint": 136, "objective": 96}[kind]
    mid = _log_int(rng, 14, top)  # the sides of one cavity are of one order of magnitude
    nx, ny, nz = (max(6, min(top, int(round(mid * math.exp(rng.uniform(-0.5, 0.5)))))) for _ in range(3))
    case = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "steps": 1}
    if kind in ("adjoint", "objective"):
        case.update(steps=_log_int(rng, 20, 200), probes=rng.randint(1, 24), medium="random")
        return case
    storage = "f32" if kind == "monitor" else rng.choice(["f32", "f32", "f32", "f32", "f16", "bf16", "f16c", "bf16c"])
    rect = rng.random() < 0.15
    case.update(medium=rng.choice(["vacuum", "spheres", "spheres", "random", "both"]), storage=storage,
                dy=round(rng.uniform(0.6, 1.5), 3) if rect else 0.0, dz=round(rng.uniform(0.6, 1.5), 3) if rect else 0.0)
    if kind == "monitor":
        case.update(steps=rng.randint(1, 12), reads=rng.randint(2, 10))
    else:
        # at most the largest listed case's cell updates; small cavities a few hundred steps
        most = min(300, int(512 ** 3 * 60 / (nx * ny * nz)))
        case["steps"] = _log_int(rng, 4, max(8, most))
    return case


# ------------------------------------------------------------------------------ inputs


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & (2 ** 62 - 1))
    return g


def _fields(case, seed):
    """E ~ U[-1, 1], H = 0 (the cavity workloads' initial state) in FP32 on the GPU."""
    g = _gen(seed, 1)
    sh = P.field_shapes(case["nx"], case["ny"], case["nz"])
    e = [torch.rand(s, generator=g, device=DEV) * 2.0 - 1.0 for s in sh[:3]]
    return e + [torch.zeros(s, device=DEV) for s in sh[3:]]


def _cells(case, seed, salt, lo, hi):
    s = (case["nz"], case["ny"], case["nx"])
    return torch.rand(s, generator=_gen(seed, salt), device=DEV, dtype=torch.float64) * (hi - lo) + lo


def _materials(case, seed):
    """(eps_r, mu_r) per cell in FP64 on the GPU, None where it is 1 everywhere."""
    m = case["medium"]
    if m == "vacuum":
        return None, None
    if m == "random":
        return _cells(case, seed, 2, 1.0, 4.0), None
    if m == "both":
        return _cells(case, seed, 2, 1.0, 4.0), _cells(case, seed, 3, 1.0, 1.5)
    # spheres of random permittivity, 1 elsewhere
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    r = random.Random(int(seed) * 7 + 33)
    ax = [torch.arange(n, device=DEV, dtype=torch.float64) + 0.5 for n in (nx, ny, nz)]
    inside = torch.zeros((nz, ny, nx), dtype=torch.bool, device=DEV)
    n = min(nx, ny, nz)
    for _ in range(32):
        c = [r.uniform(0, q) for q in (nx, ny, nz)]
        rad = r.uniform(n / 32, n / 8)
        d2 = [(a - q) ** 2 for a, q in zip(ax, c)]
        inside |= (d2[2][:, None, None] + d2[1][None, :, None]) + d2[0][None, None, :] < rad * rad
    eps = _cells(case, seed, 2, 1.0, 4.0)
    eps[~inside] = 1.0
    return eps, None


def _spacing(case):
    dy, dz = case.get("dy", 0.0) or 1.0, case.get("dz", 0.0) or 1.0
    return dy, dz, 0.5 / math.sqrt(1.0 + 1.0 / dy ** 2 + 1.0 / dz ** 2)


def _nodes(case, seed, count):
    """Distinct interior Ez nodes: the source first, then the probes."""
    r = random.Random(int(seed) * 13 + 5)
    got = []
    while len(got) < count + 1:
        q = (2, r.randrange(1, case["nx"]), r.randrange(1, case["ny"]), r.randrange(0, case["nz"]))
        if q not in got:
            got.append(q)
    return got[0], got[1:]


def _wave(case):
    n = np.arange(1, case["steps"] + 1)
    w = max(4.0, case["steps"] / 25.0)
    return np.exp(-((n - 3 * w) / w) ** 2)


def _requests(case, seed):
    r = random.Random(case["mix"])
    dims = list(range(case["lo"], case["hi"] + 1, 16))
    return [(r.choice(dims), r.choice(dims), r.choice(dims), r.randint(100, 400), int(seed) * 64 + q)
            for q in range(case["requests"])]


def _host(t):
    return None if t is None else t.cpu().numpy()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "pool":
        return {"kind": kind, "pool": P.Pool(4 << 30), "requests": _requests(case, seed)}
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    eps, mu = _materials(case, seed)
    if kind == "objective":
        src, probes = _nodes(case, seed, case["probes"])
        return {"kind": kind, "eps": eps.float().requires_grad_(True),
                "problem": {"nsteps": case["steps"], "src": src, "wave": _wave(case), "probes": probes}}
    if kind == "adjoint":
        src, probes = _nodes(case, seed, case["probes"])
        solver = P.Solver(nx, ny, nz, 1.0, COURANT, eps_r=_host(eps))
        solver.set_fields([np.zeros(s, np.float32) for s in P.field_shapes(nx, ny, nz)[:3]])
        return {"kind": kind, "solver": solver, "adjoint": Adjoint(solver, src, _wave(case), probes, case["steps"])}
    _, _, dt = _spacing(case)
    solver = P.Solver(nx, ny, nz, 1.0, dt, eps_r=_host(eps), mu_r=_host(mu), storage=case["storage"],
                      dy=case["dy"] or None, dz=case["dz"] or None)
    fields = _fields(case, seed)
    state = {"kind": kind, "solver": solver, "steps": case["steps"], "reads": case.get("reads", 0)}
    if kind == "roundtrip":
        host = [_host(t) for t in fields]
        state["e"], state["h"] = host[:3], host[3:]
        return state
    torch.cuda.synchronize()  # the solver's stream is its own
    solver.set_fields_device(fields)
    solver.sync()
    state["out"] = fields  # the program's tensors, filled again by every pass
    return state


def run(state):
    kind = state["kind"]
    if kind == "pool":
        pool, reqs = state["pool"], state["requests"]
        ids = [pool.submit(nx, ny, nz, n, seed=s, keep=True) for nx, ny, nz, n, s in reqs]
        pool.wait(-1)
        got = [pool.fetch(q, *r[:3], dtype=np.float32) for q, r in zip(ids, reqs)]
        for q in ids:
            pool.release(q)
        return got
    if kind == "objective":
        state["eps"].grad = None
        j = probe_objective(state["eps"], **state["problem"])
        j.backward()
        return [j.detach(), state["eps"].grad]
    if kind == "adjoint":
        j = state["adjoint"].forward()
        return [j, state["adjoint"].backward()]
    solver = state["solver"]
    if kind == "roundtrip":
        solver.set_fields(state["e"], state["h"])
        solver.step(state["steps"])
        return list(solver.get_fields(np.float32))
    if kind == "monitor":
        seen = []
        for _ in range(state["reads"]):
            solver.step(state["steps"])
            seen.append(solver.diag())
        solver.get_fields_device(state["out"])
        return {"diag": seen, "fields": state["out"]}
    solver.step(state["steps"])
    solver.get_fields_device(state["out"])
    return state["out"]


_BYTES = {"f32": 24, "f16": 12, "bf16": 12, "f16c": 20, "bf16c": 20}  # six components of a cell


def work(case):
    """Each input read once and each output written once; 30 operations a cell and step (six
    components of four additions, a difference pair and a multiply-add)."""
    kind = case["kind"]
    if kind == "pool":
        cells = [(nx * ny * nz, n) for nx, ny, nz, n, _ in _requests(case, 0)]
        return {"bytes": sum(24 * c for c, _ in cells), "flops": sum(30.0 * c * n for c, n in cells)}
    cells, n = case["nx"] * case["ny"] * case["nz"], case["steps"]
    if kind in ("adjoint", "objective"):
        # forward and reverse steps, and the gradient terms (three products and sums of five operations)
        return {"bytes": 12 * cells + 8 * cells, "flops": (30.0 + 36.0 + 21.0) * cells * n}
    state = _BYTES[case["storage"]] * cells
    rect = case["dy"] or case["dz"]
    ce = 12 * cells if case["medium"] != "vacuum" or rect else 0
    ch = 12 * cells if case["medium"] == "both" or rect else 0
    if kind == "monitor":
        # the diagnostics need the whole state and both coefficients after every few steps
        return {"bytes": case["reads"] * (2 * state + 2 * (ce + ch) + state) + 24 * cells,
                "flops": case["reads"] * (30.0 * n + 60.0) * cells}
    out = 24 * cells * (2 if kind == "roundtrip" else 1)
    return {"bytes": 2 * state + ce + ch + out, "flops": 30.0 * cells * n}


# ------------------------------------------------------------------------- 64-bit reference


def _d(a, axis):
    """Forward difference along x (2), y (1) or z (0)."""
    n = a.shape[axis]
    return a.narrow(axis, 1, n - 1) - a.narrow(axis, 0, n - 1)


def _inner(a, axes):
    for q in axes:
        a = a.narrow(q, 1, a.shape[q] - 2)
    return a


_FIXED = ((0, 1), (0, 2), (1, 2))  # axes along which Ex, Ey, Ez end on walls they are tangential to


def _curl_e(e, d):
    """The H updates' differences on every H node; d: spacings along x, y, z."""
    x, y, z = e
    return (_d(y, 0) / d[2] - _d(z, 1) / d[1], _d(z, 2) / d[0] - _d(x, 0) / d[2], _d(x, 1) / d[1] - _d(y, 2) / d[0])


def _curl_h(h, d):
    """The E updates' differences on the E nodes off the walls."""
    x, y, z = h
    return (_d(_inner(z, (0,)), 1) / d[1] - _d(_inner(y, (1,)), 0) / d[2],
            _d(_inner(x, (2,)), 0) / d[2] - _d(_inner(z, (0,)), 2) / d[0],
            _d(_inner(y, (1,)), 2) / d[0] - _d(_inner(x, (2,)), 1) / d[1])


def _ce(eps, dt):
    """dt / eps on the E nodes off the walls: the mean of the four cells that share the edge."""
    if eps is None:
        return (dt, dt, dt)
    got = []
    for a, b in _FIXED:
        m = eps
        for q in (a, b):
            m = (m.narrow(q, 0, m.shape[q] - 1) + m.narrow(q, 1, m.shape[q] - 1)) / 2
        got.append(dt / m)
    return tuple(got)


def _ch(mu, dt):
    """dt / mu on every H node: the mean of the face's two cells (wall faces: their one cell; their H stays)."""
    if mu is None:
        return (dt, dt, dt)
    got = []
    for q in (2, 1, 0):
        n = mu.shape[q]
        ext = torch.cat([mu.narrow(q, 0, 1), mu, mu.narrow(q, n - 1, 1)], q)
        got.append(dt / ((ext.narrow(q, 0, n + 1) + ext.narrow(q, 1, n + 1)) / 2))
    return tuple(got)


def _close_walls(e):
    for c, axes in zip(e, _FIXED):
        for q in axes:
            c.select(q, 0).zero_()
            c.select(q, c.shape[q] - 1).zero_()


def _step(e, h, ce, ch, d):
    for c, k, u in zip(h, ch, _curl_e(e, d)):
        c += k * u
    for c, k, u, axes in zip(e, ce, _curl_h(h, d), _FIXED):
        v = _inner(c, axes)
        v += k * u


def _exact_fields(case, seed):
    dy, dz, dt = _spacing(case)
    eps, mu = _materials(case, seed)
    f = [t.double() for t in _fields(case, seed)]
    _close_walls(f[:3])
    return f[:3], f[3:], _ce(eps, dt), _ch(mu, dt), (1.0, dy, dz)


def _exact_gradient(case, seed, eps):
    """J and dJ/d eps_r: reverse mode written out (the E curl is minus the H curl's transpose)."""
    d, dt, n = (1.0, 1.0, 1.0), COURANT, case["steps"]
    src, probes = _nodes(case, seed, case["probes"])
    wave = _wave(case)
    ce = _ce(eps, dt)
    sh = P.field_shapes(case["nx"], case["ny"], case["nz"])
    zeros = lambda q: [torch.zeros(s, device=DEV, dtype=torch.float64) for s in q]  # noqa: E731
    e, h = zeros(sh[:3]), zeros(sh[3:])
    at = [torch.tensor([p[q] for p in probes], device=DEV) for q in (3, 2, 1)]
    hist, rec = [], []
    for q in range(n):
        _step(e, h, ce, (dt,) * 3, d)
        e[2][src[3], src[2], src[1]] += float(wave[q])
        hist.append([c.clone() for c in h])
        rec.append(e[2][at[0], at[1], at[2]].clone())
    j = float(sum((r * r).sum() for r in rec))
    lam, mu, g = zeros(sh[:3]), zeros(sh[3:]), [torch.zeros_like(c) for c in ce]
    lam[2].index_put_(at, 2 * rec[-1], accumulate=True)
    for q in range(n - 1, -1, -1):
        w = zeros(sh[:3])
        for c, k, v, axes in zip(w, ce, lam, _FIXED):
            _inner(c, axes).copy_(k * _inner(v, axes))
        for c, u in zip(mu, _curl_e(w, d)):
            c -= u
        for c, v, u, axes in zip(g, lam, _curl_h(hist.pop(), d), _FIXED):
            c += _inner(v, axes) * u
        for v, u, axes in zip(lam, _curl_h([dt * c for c in mu], d), _FIXED):
            t = _inner(v, axes)
            t -= u
        if q:
            lam[2].index_put_(at, 2 * rec[q - 1], accumulate=True)
    out = torch.zeros_like(eps)
    for c, k, (a, b) in zip(g, ce, _FIXED):
        t = -c * k * k / (4 * dt)  # to each of the edge's four cells
        for p in (0, 1):
            for q in (0, 1):
                v = out.narrow(a, p, out.shape[a] - 1).narrow(b, q, out.shape[b] - 1)
                v += t
    return j, out


def _mix(z):
    """SplitMix64's output function on int64 tensors."""
    shr = lambda v, n: (v >> n) & ((1 << (64 - n)) - 1)  # noqa: E731
    z = (z ^ shr(z, 30)) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ shr(z, 27)) * (0x94D049BB133111EB - (1 << 64))
    return z ^ shr(z, 31)


def _seeded(nx, ny, nz, seed):
    """The seeded initial state: counter (component << 40) + linear index, u = (output >> 11) 2^-53, E = 2u - 1."""
    sh = P.field_shapes(nx, ny, nz)
    e = []
    for f, s in enumerate(sh[:3]):
        c = torch.arange(math.prod(s), device=DEV, dtype=torch.int64) + ((f << 40) + 1)
        z = _mix(c * (0x9E3779B97F4A7C15 - (1 << 64)) + seed)
        u = ((z >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53
        e.append((2 * u - 1).float().double().reshape(s))
    return e, [torch.zeros(s, device=DEV, dtype=torch.float64) for s in sh[3:]]


def exact(case, seed):
    kind = case["kind"]
    one = (1.0, 1.0, 1.0)
    if kind == "pool":
        got = []
        for nx, ny, nz, n, s in _requests(case, seed):
            e, h = _seeded(nx, ny, nz, s)
            _close_walls(e)
            for _ in range(n):
                _step(e, h, (COURANT,) * 3, (COURANT,) * 3, one)
            got.append([c.cpu() for c in e + h])
        return got
    if kind == "adjoint":
        j, g = _exact_gradient(case, seed, _materials(case, seed)[0])
        return [j, g.cpu().numpy()]
    if kind == "objective":
        eps = _materials(case, seed)[0].float().double()
        j, g = _exact_gradient(case, seed, eps)
        return [torch.tensor(j, dtype=torch.float64), g]
    e, h, ce, ch, d = _exact_fields(case, seed)
    if kind != "monitor":
        for _ in range(case["steps"]):
            _step(e, h, ce, ch, d)
        return e + h
    seen = []
    for _ in range(case["reads"]):
        for _ in range(case["steps"]):
            _step(e, h, ce, ch, d)
        # rectangular cells report the stored variables (see fdtd.h): no plain value for those
        plain = not (case["dy"] or case["dz"])
        seen.append({"energy": None, "max_div_b": None, "max_e_tan": None, "nonfinite": 0.0,
                     "sum_e2": float(sum((c * c).sum() for c in e)) if plain else None,
                     "sum_h2": float(sum((c * c).sum() for c in h)) if plain else None})
    return {"diag": seen, "fields": e + h}
