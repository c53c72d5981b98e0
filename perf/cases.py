"""Workloads of the solver for timing and for comparing results.

A case is one stretch of a simulation as a program drives it: a box (or an
ensemble of boxes) that exists already is advanced by a number of RK3 steps, in
most cases with the global diagnostics of every step, and its state is then
fetched as a snapshot.  The kernel shape is the library's own choice.  A box
carries its state from one pass to the next, as a time loop does.

A single-precision run keeps its record (snapshot and diagnostics) in single
precision, the precision its state is stored in.

listed() are the cases themselves, draw() gives others of the same ranges:
edges of 24 to 512 points, equal or not, multiples of a tile or not; FP64, FP32
and FP32 with FP64 RK3 arithmetic; the 55- and the 19-point method; both state
layouts; launch by launch or replayed from captured graphs; with and without
the external force; ensembles of 4 to 12 boxes.

exact() is the same computation written plainly in 64 bits: the sixth-order
differences of the paper's Sec. 2.3 on periodically padded arrays and the
2N-storage RK3 of Sec. 2.4.
"""
import math

import numpy as np
import torch

import paper_1707_08900_amd as fd6

TWO_PI = 2.0 * math.pi
DEVICE = "cuda:0"
EDGES = (96, 32, 64, 48)  # of an ensemble's boxes, in turn
MAX_COST = 512 ** 3 * 10 * 32  # points x steps x bytes of a point's state, in and out


def _box(name, shape, precision, steps, *, variant="55p", layout="soa", diag="step", graph=False,
         force=False, amplitude=0.1, kmax=16.0, nu=1e-3):
    """diag: "step" (after every step), "end" (after the last one) or "none"."""
    nz, ny, nx = shape
    return {"name": name, "kind": "box", "nz": nz, "ny": ny, "nx": nx, "precision": precision,
            "variant": variant, "layout": layout, "steps": steps, "diag": diag, "graph": graph,
            "force": force, "amplitude": amplitude, "kmax": kmax, "nu": nu}


def listed():
    return [
        # one step of the smallest box that is run in earnest: launches and latency
        _box("step_32_fp32", (32, 32, 32), "fp32", 1, amplitude=1e-2, kmax=4.0, nu=5e-3),
        # a small double-precision reference run, replayed from captured graphs
        _box("run_64_fp64_graph", (64, 64, 64), "fp64", 20, diag="end", graph=True,
             amplitude=1e-2, kmax=8.0, nu=2e-3),
        # the validation size of the paper's methods, a step at a time
        _box("run_128_fp32_aos", (128, 128, 128), "fp32", 20, layout="aos", amplitude=1e-2,
             kmax=8.0, nu=2e-3),
        # a box that fills no tile, in the default layout
        _box("run_ragged_fp32", (101, 75, 150), "fp32", 10, amplitude=2e-2, kmax=6.0, nu=3e-3),
        # an ordinary production box
        _box("run_256_fp32_aos", (256, 256, 256), "fp32", 10, layout="aos"),
        # single precision in the default layout
        _box("run_384_fp32_soa", (384, 384, 384), "fp32", 5),
        # the throughput box of the benchmark
        _box("run_512_fp32_aos", (512, 512, 512), "fp32", 10, layout="aos"),
        # the same in double precision
        _box("run_512_fp64_aos", (512, 512, 512), "fp64", 4, layout="aos"),
        # single-precision state with the time integration in double precision
        _box("run_320_fp32_acc64_aos", (320, 320, 320), "fp32_acc64", 5, layout="aos"),
        # forced turbulence: the 19-point method with a new force in every step
        _box("forced_256_19p_fp32", (256, 256, 256), "fp32", 10, variant="19p", diag="none",
             force=True),
        # the 19-point method in double precision on a box of unequal edges
        _box("run_240_19p_fp64", (192, 240, 300), "fp64", 5, variant="19p", nu=2e-3),
        # a parameter study: uneven boxes advanced together, results fetched to the host
        {"name": "ensemble_12_fp32_aos", "kind": "ensemble", "boxes": 12, "precision": "fp32",
         "layout": "aos", "steps": 100},
    ]


def draw(rng):
    def edge(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n // 16 * 16 if n >= 32 and rng.random() < 0.35 else n

    if rng.random() < 0.12:
        return {"kind": "ensemble", "boxes": rng.randint(4, 12),
                "precision": rng.choice(["fp32", "fp64"]), "layout": rng.choice(["soa", "aos"]),
                "steps": rng.randint(10, 60)}
    if rng.random() < 0.5:
        n = edge(24, 512)
        shape = (n, n, n)
    else:
        shape = (edge(24, 512), edge(24, 512), edge(24, 512))
    precision = rng.choice(["fp32", "fp32", "fp64", "fp32_acc64"])
    variant = rng.choice(["55p", "55p", "19p"])
    layout = "soa" if variant == "19p" else rng.choice(["soa", "aos"])
    points = shape[0] * shape[1] * shape[2]
    most = MAX_COST // (points * (64 if precision == "fp64" else 32))
    steps = max(1, min(rng.randint(1, 30), int(0.8 * most)))
    h = TWO_PI / min(shape)
    amplitude = rng.choice([1e-2, 3e-2, 1e-1])
    # captured steps record where their diagnostics go, so a replaying program
    # asks for them at the end
    graph = rng.random() < 0.3
    diag = rng.choice(["end", "none"]) if graph else rng.choice(["step", "step", "end", "none"])
    return {"kind": "box", "nz": shape[0], "ny": shape[1], "nx": shape[2],
            "precision": precision, "variant": variant, "layout": layout, "steps": steps,
            "diag": diag, "graph": graph,
            "force": rng.random() < 0.2, "amplitude": amplitude,
            "kmax": min(16.0, min(shape) / 8.0), "nu": max(1e-3, 0.3 * amplitude * h)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _waves(n, k, device):
    j = torch.arange(n, dtype=torch.int64)
    ang = torch.remainder(k[:, None] * j[None, :], n).double() * (TWO_PI / n)
    return torch.polar(torch.ones_like(ang), ang).to(device)


def _fourier_field(shape, gen, amplitude, kmax, modes=16):
    """Sum of random-phase Fourier modes with 1 <= |k| <= kmax."""
    nz, ny, nx = shape
    m = max(1, int(kmax))
    ks = torch.zeros(0, 3, dtype=torch.int64)
    while len(ks) < modes:
        k = torch.randint(-m, m + 1, (4 * modes, 3), generator=gen)
        n2 = (k * k).sum(1)
        ks = torch.cat([ks, k[(n2 > 0) & (n2 <= kmax * kmax)]])
    ks = ks[:modes]
    ph = torch.rand(modes, generator=gen, dtype=torch.float64) * TWO_PI
    ex, ey, ez = (_waves(n, ks[:, a], DEVICE) for a, n in ((0, nx), (1, ny), (2, nz)))
    ez = ez * torch.polar(torch.ones_like(ph), ph).to(DEVICE)[:, None]
    zy = (ez[:, :, None] * ey[:, None, :]).reshape(modes, nz * ny).t()
    a = torch.cat([zy.real, -zy.imag], 1).contiguous()
    b = torch.cat([ex.real, ex.imag], 0).contiguous()
    return (a @ b).reshape(nz, ny, nx).mul_(amplitude / math.sqrt(modes))


def _fields(shape, seed, amplitude, kmax, precision):
    """lnrho, ux, uy, uz on the device in FP64, representable in the state's precision."""
    gen = torch.Generator().manual_seed(int(seed))
    f = [_fourier_field(shape, gen, amplitude, kmax) for _ in range(4)]
    return f if precision == "fp64" else [x.float().double() for x in f]


def _params(shape, fields, nu, cs=1.0):
    nz, ny, nx = shape
    dx, dy, dz = TWO_PI / nx, TWO_PI / ny, TWO_PI / nz
    _, ux, uy, uz = fields
    umax = math.sqrt(float((ux * ux + uy * uy + uz * uz).max()))
    return nu, cs, dx, dy, dz, 0.4 * min(dx, dy, dz) / (cs + umax)


def _forces(seed, count):
    """One random mode per step: k from 1 <= |k| <= 3, e perpendicular to it, a phase."""
    rng = np.random.default_rng(int(seed) + 77)
    r = np.arange(-3, 4)
    k = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3).astype(float)
    kk = np.linalg.norm(k, axis=1)
    k = k[(kk >= 1.0) & (kk <= 3.0)]
    out = []
    for _ in range(count):
        v = k[rng.integers(len(k))]
        e = np.cross(v, rng.normal(size=3))
        e /= np.linalg.norm(e)
        out.append({"k": tuple(float(x) for x in v), "e": tuple(float(x) for x in e), "f0": 0.02,
                    "phase": float(rng.uniform(0.0, TWO_PI))})
    return out


def _members(case, seed):
    """(edge, amplitude, nu, fields) of every box of an ensemble."""
    rng = np.random.default_rng(int(seed))
    out = []
    for b in range(case["boxes"]):
        n = EDGES[b % 4]
        amplitude, nu = float(rng.uniform(1e-3, 5e-2)), float(rng.uniform(2e-3, 1e-2))
        f = _fields((n, n, n), 1000 * int(seed) + b, amplitude, n / 8.0, case["precision"])
        out.append((n, amplitude, nu, f))
    return out


def _shape(case):
    return case["nz"], case["ny"], case["nx"]


def prepare(case, seed):
    if case["kind"] == "ensemble":
        members = _members(case, seed)
        batch = fd6.Batch([(n, n, n) for n, _, _, _ in members], case["precision"],
                          layout=case["layout"])
        batch.set_params([_params((n, n, n), f, nu) for n, _, nu, f in members])
        for i, (_, _, _, f) in enumerate(members):
            batch.init_fields(i, [x.cpu().numpy() for x in f])
        return {"case": case, "batch": batch}
    shape = _shape(case)
    fields = _fields(shape, seed, case["amplitude"], case["kmax"], case["precision"])
    box = fd6.Box(shape, case["precision"], case["variant"], layout=case["layout"])
    box.set_params(*_params(shape, fields, case["nu"]))
    box.set_graph(case["graph"])
    box.init_fields(fields)
    diag = torch.zeros(case["steps"], 5, dtype=torch.float64, device=DEVICE)
    return {"case": case, "box": box, "diag": diag,
            "forces": _forces(seed, case["steps"]) if case["force"] else None}


def run(state):
    case = state["case"]
    if case["kind"] == "ensemble":
        batch = state["batch"]
        batch.step(case["steps"])
        out = [f for i in range(batch.n) for f in batch.get_fields(i)]
        return out if case["precision"] == "fp64" else [f.astype(np.float32) for f in out]
    box, diag, steps = state["box"], state["diag"], case["steps"]
    if state["forces"] is not None or case["diag"] == "step":
        for s in range(steps):
            if state["forces"] is not None:
                box.set_forcing(state["forces"][s])
            if case["diag"] == "step" or (case["diag"] == "end" and s == steps - 1):
                box.step_reduce(1, diag[s])
            else:
                box.step(1)
    elif case["diag"] == "end":
        box.step_reduce(steps, diag[steps - 1])
    else:
        box.step(steps)
    fields = box.get_fields_device()
    if case["precision"] == "fp64":
        return {"fields": fields, "diag": diag.clone()}
    return {"fields": [f.float() for f in fields], "diag": diag.float()}


def work(case):
    """Every substep reads the state once and writes it once; the snapshot is
    read and written once.  Additions and multiplications of the stencils (12
    first, 9 second and 6 mixed derivatives, or the 3 of the divergence), of the
    right-hand side and of the update."""
    es = 8 if case["precision"] == "fp64" else 4
    if case["kind"] == "ensemble":
        points = sum(EDGES[b % 4] ** 3 for b in range(case["boxes"]))
        ops = 354
    else:
        points = case["nz"] * case["ny"] * case["nx"]
        ops = 354 if case["variant"] == "55p" else 300
    steps = case["steps"]
    return {"bytes": points * 4 * es * (2 * 3 * steps + 2), "flops": points * ops * 3 * steps}


# ---------------------------------------------------------------------------
# The same in 64 bits, without the library
# ---------------------------------------------------------------------------
_W1 = (45.0, -9.0, 1.0)          # / 60 h
_W2 = (270.0, -27.0, 2.0)        # centre -490, / 180 h^2; mixed / 720 h h
_ALPHA = (0.0, -5.0 / 9.0, -153.0 / 128.0)
_BETA = (1.0 / 3.0, 15.0 / 16.0, 8.0 / 15.0)
_AXIS = {0: 2, 1: 1, 2: 0}       # x, y, z -> array dimension


def _pad(f):
    for d in range(3):
        n = f.shape[d]
        f = torch.cat([f.narrow(d, n - 3, 3), f, f.narrow(d, 0, 3)], d)
    return f


def _at(p, **shift):
    """The view of a padded array shifted by the given numbers of points along x, y, z."""
    for i, name in enumerate("xyz"):
        d = _AXIS[i]
        p = p.narrow(d, 3 + shift.get(name, 0), p.shape[d] - 6)
    return p


def _d1(p, a, h):
    c = "xyz"[a]
    out = None
    for k in (1, 2, 3):
        t = (_at(p, **{c: k}) - _at(p, **{c: -k})).mul_(_W1[k - 1] / (60.0 * h[a]))
        out = t if out is None else out.add_(t)
    return out


def _lap_add(out, p, a, h, scale):
    c = "xyz"[a]
    s = scale / (180.0 * h[a] * h[a])
    out.add_(_at(p), alpha=-490.0 * s)
    for k in (1, 2, 3):
        out.add_(_at(p, **{c: k}), alpha=_W2[k - 1] * s)
        out.add_(_at(p, **{c: -k}), alpha=_W2[k - 1] * s)


def _mixed_add(out, p, a, b, h, scale):
    c, d = "xyz"[a], "xyz"[b]
    s = scale / (720.0 * h[a] * h[b])
    for k in (1, 2, 3):
        out.add_(_at(p, **{c: k, d: k}) - _at(p, **{c: -k, d: k}), alpha=_W2[k - 1] * s)
        out.add_(_at(p, **{c: -k, d: -k}) - _at(p, **{c: k, d: -k}), alpha=_W2[k - 1] * s)


def _rhs(f, nu, cs, h, variant, force):
    pads = [_pad(x) for x in f]
    g = [_d1(pads[0], a, h) for a in range(3)]
    J = [[_d1(pads[1 + i], a, h) for a in range(3)] for i in range(3)]
    div = J[0][0] + J[1][1] + J[2][2]
    u = f[1:]
    r = [-(u[0] * g[0] + u[1] * g[1] + u[2] * g[2]) - div]
    dpad = _pad(div) if variant == "19p" else None
    for i in range(3):
        out = g[i] * (-cs * cs)
        for j in range(3):
            out.sub_(u[j] * J[i][j])
            out.add_((J[i][j] + J[j][i]).mul_(g[j]), alpha=nu)
        out.add_(div * g[i], alpha=-2.0 * nu / 3.0)
        third = nu / 3.0
        for a in range(3):
            _lap_add(out, pads[1 + i], a, h, nu + (third if a == i and variant == "55p" else 0.0))
        if variant == "19p":
            out.add_(_d1(dpad, i, h), alpha=third)
        else:
            for j in range(3):
                if j != i:
                    _mixed_add(out, pads[1 + j], min(i, j), max(i, j), h, third)
        if force is not None:
            out.add_(force[1], alpha=force[0][i])
        r.append(out)
    return r


def _force(draw_, shape, h, cs, dt):
    k, e = np.array(draw_["k"]), np.array(draw_["e"])
    kk, ke = math.sqrt(float(k @ k)), float(k @ e)
    a = draw_["f0"] * cs * math.sqrt(kk * cs / dt) * np.cross(k, e) / math.sqrt(kk * kk - ke * ke)
    x, y, z = (torch.arange(n, dtype=torch.float64, device=DEVICE) * h[i]
               for i, n in ((0, shape[2]), (1, shape[1]), (2, shape[0])))
    ang = (float(k[2]) * z + draw_["phase"])[:, None, None] + (float(k[1]) * y)[None, :, None]
    return a, torch.cos(ang + (float(k[0]) * x)[None, None, :])


def _step(f, nu, cs, h, dt, variant, force):
    w = None
    for s in range(3):
        r = _rhs(f, nu, cs, h, variant, force)
        w = [x * dt for x in r] if w is None else [y.mul_(_ALPHA[s]).add_(x, alpha=dt)
                                                   for x, y in zip(r, w)]
        f = [x.add(y, alpha=_BETA[s]) for x, y in zip(f, w)]
    return f


def _diag(f, h):
    rho, u2 = torch.exp(f[0]), f[1] * f[1] + f[2] * f[2] + f[3] * f[3]
    dv = h[0] * h[1] * h[2]
    return torch.stack([rho.sum() * dv, (rho * u2).sum() * (0.5 * dv), f[0].sum(),
                        u2.max().sqrt(), torch.zeros((), dtype=torch.float64, device=DEVICE)])


def exact(case, seed):
    if case["kind"] == "ensemble":
        out = []
        for n, _, nu, f in _members(case, seed):
            p = _params((n, n, n), f, nu)
            for _ in range(case["steps"]):
                f = _step(f, p[0], p[1], p[2:5], p[5], "55p", None)
            out += [x.cpu().numpy() for x in f]
        return out
    shape = _shape(case)
    f = _fields(shape, seed, case["amplitude"], case["kmax"], case["precision"])
    nu, cs, dx, dy, dz, dt = _params(shape, f, case["nu"])
    h = (dx, dy, dz)
    diag = torch.zeros(case["steps"], 5, dtype=torch.float64, device=DEVICE)
    forces = _forces(seed, case["steps"]) if case["force"] else None
    for s in range(case["steps"]):
        force = _force(forces[s], shape, h, cs, dt) if forces else None
        f = _step(f, nu, cs, h, dt, case["variant"], force)
        if case["diag"] == "step" or (case["diag"] == "end" and s == case["steps"] - 1):
            diag[s] = _diag(f, h)
    return {"fields": f, "diag": diag}
