"""The measured work: steps, diagnostics and gradients of the WENO5-CT MHD framework on one GPU.

A case names one path through the public entry points (``binding.Patch``,
``binding.step_static``, ``rollout.rollout``) with a box size and the options of
``binding.config``.  Inputs are smooth random periodic fields (a few plane waves
per component over a uniform background), made on the GPU from the seed alone.

Paths:
  step      ``Patch.step``: one time step, its dt taken on the device
  static    ``step_static``: one step of caller-owned tensors without a patch
  graph     ``Patch.capture(4)`` once, then its ``replay()``
  monitor   ``Patch.compute_dt`` and ``Patch.diagnostics``, read by the host
  adjoint   ``Patch.adjoint_step``: the cotangents of one recorded step
  gradient  ``rollout``: forward, backward and the gradients of A and v

``exact`` computes the same results with plain torch operations in 64 bits
(gradients by autograd through them).
"""
import math

import torch
from torch.utils.checkpoint import checkpoint

from paper_1812_04278_amd import binding, rollout

DEV = "cuda"
GAMMA = 5.0 / 3.0
CFL = {"ssprk3": 0.4, "rk4": 0.8}
GRAPH_STEPS = 4
RHO_FLOOR, P_FLOOR = 1e-3, 1e-4

PRECISION = {"fp64": binding.WM_FP64, "mixed": binding.WM_MIXED, "fp32": binding.WM_MIXED_F32STATE}
WEIGHTS = {"js": binding.WM_WENO_JS, "z": binding.WM_WENO_Z}
INTEGRATOR = {"ssprk3": binding.WM_SSPRK3, "rk4": binding.WM_RK4}


def _case(path, nx, ny, nz, mach, name=None, **options):
    c = dict(path=path, nx=nx, ny=ny, nz=nz, mach=mach, precision="fp64", weights="js", integrator="ssprk3", walls="",
             floors=False, steps=1)
    c.update(options)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a tight loop over a tiny box without an allocator: launches and latency
        _case("static", 16, 16, 16, 0.1, name="static 16"),
        # the small throughput workload: a box far below what fills the chip
        _case("step", 32, 32, 32, 0.1, name="step 32"),
        # a small box stepped by graph replays, WENO-Z
        _case("graph", 48, 40, 36, 0.5, name="graph 48x40x36 weno-z", weights="z"),
        # an ordinary box with odd sizes along every axis
        _case("step", 97, 75, 61, 0.5, name="step 97x75x61"),
        # reflecting walls along x and z with the protection floors
        _case("step", 120, 90, 80, 0.8, name="walls 120x90x80", walls="xz", floors=True),
        # the four-stage integrator with the sharper weights on a medium box
        _case("step", 128, 128, 128, 1.0, name="rk4 weno-z 128", weights="z", integrator="rk4"),
        # the throughput workload: Mach 2, all in double precision
        _case("step", 256, 256, 256, 2.0, name="step 256"),
        # the mixed-precision workload: double state, single-precision characteristic work
        _case("step", 256, 256, 256, 0.1, name="mixed 256", precision="mixed"),
        # the large turbulence box, single-precision state
        _case("step", 512, 512, 512, 5.0, name="fp32 state 512", precision="fp32"),
        # what a production loop reads every few steps: dt, totals, divergence, minima
        _case("monitor", 256, 256, 256, 2.0, name="monitor 256"),
        # the cotangents of one step with recorded stages: the backward pass's unit of work
        _case("adjoint", 128, 128, 128, 1.0, name="adjoint step 128"),
        # a whole gradient of a small control problem: forward, recomputation, backward
        _case("gradient", 48, 48, 48, 1.0, name="gradient 48, 6 steps", steps=6),
    ]


def _sizes(rng, lo, hi):
    """Three sizes around one drawn over its logarithm; about half of them odd."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return [max(12, min(hi, int(round(n * rng.uniform(0.75, 1.0))) + rng.randrange(2))) for _ in range(3)]


def draw(rng):
    path = rng.choice(["step", "step", "step", "static", "graph", "monitor", "adjoint", "gradient"])
    lo, hi = {"step": (20, 288), "static": (12, 56), "graph": (20, 96), "monitor": (32, 288), "adjoint": (24, 144),
              "gradient": (16, 72)}[path]
    nx, ny, nz = _sizes(rng, lo, hi)
    c = _case(path, nx, ny, nz, round(rng.uniform(0.1, 1.0), 2))
    c["weights"] = rng.choice(["js", "js", "z"])
    if path in ("step", "graph", "static", "monitor"):
        c["precision"] = rng.choice(["fp64", "fp64", "mixed", "fp32"])
    if path in ("step", "graph", "static"):
        c["integrator"] = rng.choice(["ssprk3", "ssprk3", "rk4"])
    if path == "step":
        c["walls"] = rng.choice(["", "", "", "x", "y", "xz"])
        c["floors"] = c["integrator"] == "ssprk3" and rng.random() < 0.25
    if path == "gradient":
        c["steps"] = rng.choice([3, 4, 6])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

B0 = (1.0, 0.5, 0.25)
P0 = 0.6


def _waves(gen, shape, offset, count, kmax):
    """Sum of ``count`` plane waves with integer wave numbers up to kmax, unit variance."""
    nz, ny, nx = shape
    k = torch.randint(-kmax, kmax + 1, (count, 3), generator=gen).tolist()
    ph = (2 * math.pi * torch.rand(count, generator=gen, dtype=torch.float64)).tolist()
    am = torch.randn(count, generator=gen, dtype=torch.float64)
    am = (am / am.square().sum().mul(0.5).sqrt()).tolist()
    ax = [(torch.arange(n, device=DEV, dtype=torch.float64) + o) * (2 * math.pi / n) for n, o in zip((nx, ny, nz), offset)]
    f = torch.zeros(shape, device=DEV, dtype=torch.float64)
    for (kx, ky, kz), p, a in zip(k, ph, am):
        if kx == ky == kz == 0:
            kx = 1
        f.add_(torch.cos(ax[0] * kx + (ax[1] * ky)[:, None] + (ax[2] * kz + p)[:, None, None]), alpha=a)
    return f


def _fields(case, seed):
    """rho, v [3] on zones and A [3] on edges (A_x at (i, j+1/2, k+1/2), ...); with
    walls the tangential potential vanishes on the wall edges."""
    shape = (case["nz"], case["ny"], case["nx"])
    h = _h(case)
    gen = torch.Generator().manual_seed(int(seed))
    kmax = 8 if min(shape) >= 256 else max(1, min(4, min(shape) // 8))
    zone, edge = (0.5, 0.5, 0.5), [(0.5, 1.0, 1.0), (1.0, 0.5, 1.0), (1.0, 1.0, 0.5)]
    rho = 1.0 + 0.15 * _waves(gen, shape, zone, 6, kmax)
    v = torch.stack([0.05 * (d + 1) + case["mach"] / math.sqrt(3.0) * _waves(gen, shape, zone, 6, kmax) for d in range(3)])
    rho.clamp_(min=0.3)
    scale = 0.15 * h * max(shape) / (2 * math.pi * kmax)
    A = torch.stack([scale * _waves(gen, shape, edge[d], 6, kmax) for d in range(3)])
    for axis in _walls(case):
        for d in range(3):
            if d != axis:
                A[d].select(2 - axis, shape[2 - axis] - 1).zero_()
    return rho, v, A


def _h(case):
    return 1.0 / max(case["nx"], case["ny"], case["nz"])


def _walls(case):
    return [a for a in range(3) if "xyz"[a] in case["walls"]]


def _background(case):
    return tuple(0.0 if a in _walls(case) else b for a, b in enumerate(B0))


def _config(case):
    walls = [int(a in _walls(case)) for a in range(3)]
    floors = dict(rho_floor=RHO_FLOOR, p_floor=P_FLOOR) if case["floors"] else {}
    return binding.config(nx=case["nx"], ny=case["ny"], nz=case["nz"], h=_h(case), cfl=CFL[case["integrator"]],
                          weights=WEIGHTS[case["weights"]], precision=PRECISION[case["precision"]],
                          integrator=INTEGRATOR[case["integrator"]], walls=walls, **floors)


_stream = None


def _graph_stream():
    """The program's one stream for captured work (capture needs one that is not the default)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def _cotangents(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    gen = torch.Generator(device=DEV).manual_seed(int(seed) + 77)
    new = lambda c: torch.randn((c,) + shape, generator=gen, device=DEV, dtype=torch.float64)
    return new(5), new(3)


def prepare(case, seed):
    path = case["path"]
    rho, v, A = _fields(case, seed)
    if path == "graph":
        torch.cuda.synchronize()
    p = binding.Patch(_config(case), device=DEV, stream=_graph_stream() if path == "graph" else None)
    state = dict(path=path, patch=p, case=case)
    if path == "gradient":
        state.update(rho=rho, v=v.requires_grad_(), A=A.requires_grad_(), cot=_cotangents(case, seed))
        return state
    p.init_from_potential(rho, v, A, P0, _background(case))
    if path == "static":
        state.update(cfg=p.cfg, hydro=p.hydro, bface=p.bface, bcell=p.bcell)
    if path == "graph":
        state["graph"] = p.capture(GRAPH_STEPS)
    if path == "adjoint":
        Un = (p.hydro.clone(), p.bface.clone())
        dt = p.compute_dt()
        state.update(Un=Un, dt=dt, stages=p.step_record(dt), lam=_cotangents(case, seed))
        p._adj()
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    path, p = state["path"], state["patch"]
    if path == "step":
        p.step()
        return p.hydro, p.bface, p.bcell
    if path == "static":
        binding.step_static(state["cfg"], state["hydro"], state["bface"], state["bcell"])
        return state["hydro"], state["bface"], state["bcell"]
    if path == "graph":
        state["graph"].replay()
        return p.hydro, p.bface, p.bcell
    if path == "monitor":
        dt = p.compute_dt()
        return dict(p.diagnostics(), dt=dt)
    if path == "adjoint":
        lam_h, lam_b = (x.clone() for x in state["lam"])
        p.adjoint_step(*state["Un"], state["dt"], lam_h, lam_b, *state["stages"])
        return lam_h, lam_b
    A, v = state["A"], state["v"]
    out = rollout.rollout(A, v, state["rho"], p, state["case"]["steps"], 3, P0, B0)
    gA, gv = torch.autograd.grad(out[:2], (A, v), state["cot"])
    return out[0].detach(), out[1].detach(), gA, gv


# operations per zone: a face of a sweep takes about 2,170, its reverse about
# three times as many; the divergence, corner fluxes and the stage about 150
FACE, UPDATE = 2170, 150


def work(case):
    n = case["nx"] * case["ny"] * case["nz"]
    size = 4 if case["precision"] == "fp32" else 8
    stages = 4 if case["integrator"] == "rk4" else 3
    step = stages * (3 * FACE + UPDATE) * n
    path = case["path"]
    if path in ("step", "static"):
        return dict(bytes=(8 + 11) * size * n, flops=step)
    if path == "graph":
        return dict(bytes=(8 + 11) * size * n, flops=GRAPH_STEPS * step)
    if path == "monitor":
        return dict(bytes=11 * size * n, flops=200 * n)
    if path == "adjoint":
        return dict(bytes=(3 * 8 + 8 + 8) * 8 * n, flops=3 * step)
    return dict(bytes=(7 + 8 + 8 + 6) * 8 * n, flops=4 * case["steps"] * step)


# ---------------------------------------------------------------------------
# the same results in 64 bits with plain torch operations
# ---------------------------------------------------------------------------

def _at(f, o, axis):
    return torch.roll(f, -o, f.dim() - 1 - axis)


def _mirror(f, axis, odd=False):
    d = f.dim() - 1 - axis
    return torch.cat([f, -f.flip(d) if odd else f.flip(d)], d)


def _mirror_face(f, axis):
    d = f.dim() - 1 - axis
    n = f.shape[d]
    return torch.cat([f, -f.narrow(d, 0, n - 1).flip(d), torch.zeros_like(f.narrow(d, 0, 1))], d)


def _double(U, axis):
    """The state with its mirror image behind the upper wall of an axis."""
    rho, m, E, b = U
    return (_mirror(rho, axis), [_mirror(m[c], axis, c == axis) for c in range(3)], _mirror(E, axis),
            [_mirror_face(b[c], axis) if c == axis else _mirror(b[c], axis) for c in range(3)])


def _zone_b(b):
    return [(9.0 * (_at(b[a], -1, a) + b[a]) - (_at(b[a], -2, a) + _at(b[a], 1, a))) / 16.0 for a in range(3)]


def _zone_b_walls(b, walls):
    sizes = [b[0].shape[2 - a] for a in range(3)]
    for a in walls:
        b = [_mirror_face(b[c], a) if c == a else _mirror(b[c], a) for c in range(3)]
    B = _zone_b(b)
    for a in walls:
        B = [x.narrow(2 - a, 0, sizes[a]) for x in B]
    return B


def _pressure(U, B):
    rho, m, E, _ = U
    kin = sum(m[d] * m[d] for d in range(3)) / rho
    return (GAMMA - 1.0) * (E - 0.5 * (kin + sum(x * x for x in B)))


def _speeds(rho, Bn, Bt, P):
    """Fast, Alfven and slow speeds and the sound speed squared."""
    a2, bn2, bt2 = GAMMA * P / rho, Bn * Bn / rho, (Bt[0] * Bt[0] + Bt[1] * Bt[1]) / rho
    D = torch.sqrt((a2 - bn2 - bt2) ** 2 + 4.0 * a2 * bt2)
    cf2 = 0.5 * (a2 + bn2 + bt2 + D)
    return torch.sqrt(cf2), torch.sqrt(bn2), torch.sqrt(a2 * bn2 / cf2), a2, D


def _phi(a, b, c, d, weights):
    I = [13.0 * (a - b) ** 2 + 3.0 * (a - 3.0 * b) ** 2, 13.0 * (b - c) ** 2 + 3.0 * (b + c) ** 2,
         13.0 * (c - d) ** 2 + 3.0 * (3.0 * c - d) ** 2]
    if weights == "js":
        w = [g / (1e-6 + s) ** 2 for g, s in zip((1.0, 6.0, 3.0), I)]
    else:
        tau = (I[0] - I[2]).abs()
        w = [g * (1.0 + (tau / (1e-40 + s)) ** 2) for g, s in zip((1.0, 6.0, 3.0), I)]
    t = w[0] + w[1] + w[2]
    return w[0] / t * (a - 2.0 * b + c) / 3.0 + (w[2] / t - 0.5) * (b - 2.0 * c + d) / 6.0


def _sweep(axis, weights, rho, m, E, v, B, P):
    """Interface fluxes (rho, m_n, m_t1, m_t2, E) and the two transport fluxes of one direction."""
    n, t, s_ = axis, (axis + 1) % 3, (axis + 2) % 3
    v, m, B = [v[n], v[t], v[s_]], [m[n], m[t], m[s_]], [B[n], B[t], B[s_]]
    Pt = P + 0.5 * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2])
    vB = v[0] * B[0] + v[1] * B[1] + v[2] * B[2]
    q = [rho, m[0], m[1], m[2], B[1], B[2], E]
    F = [m[0], m[0] * v[0] + Pt - B[0] * B[0], m[0] * v[1] - B[0] * B[1], m[0] * v[2] - B[0] * B[2],
         B[1] * v[0] - B[0] * v[1], B[2] * v[0] - B[0] * v[2], (E + Pt) * v[0] - B[0] * vB]
    cf, ca, cs, _, _ = _speeds(rho, B[0], B[1:], P)
    lf = lambda x: torch.maximum(x.abs(), _at(x, 1, axis).abs())
    face = lambda x: 0.5 * (x + _at(x, 1, axis))
    alpha = [lf(v[0] - cf), lf(v[0] - ca), lf(v[0] - cs), lf(v[0]), lf(v[0] + cs), lf(v[0] + ca), lf(v[0] + cf)]
    dq, dF = [_at(x, 1, axis) - x for x in q], [_at(x, 1, axis) - x for x in F]
    # the face state and its eigenvectors
    r, u, b, p = face(rho), [face(x) for x in v], [face(x) for x in B], face(P)
    f, _, sl, a2, D = _speeds(r, b[0], b[1:], p)
    c, sr = torch.sqrt(a2), torch.sqrt(r)
    bp = torch.sqrt(b[1] * b[1] + b[2] * b[2])
    by, bz, sg = b[1] / bp, b[2] / bp, torch.where(b[0] >= 1e-30, 1.0, -1.0).to(r.dtype)
    dab, cross = a2 - (b[0] * b[0] + bp * bp) / r, 4.0 * a2 * bp * bp / r
    large, small = (D + dab.abs()) / (2.0 * D), cross / (D + dab.abs()) / (2.0 * D)
    af, as_ = torch.sqrt(torch.where(dab >= 0, large, small)), torch.sqrt(torch.where(dab >= 0, small, large))
    u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
    bu = by * u[1] + bz * u[2]
    Gf, Gs, Ga = af * f * u[0] - as_ * sl * sg * bu, as_ * sl * u[0] + af * f * sg * bu, sg * (bz * u[1] - by * u[2])
    k, g1 = 0.5 / a2, 1.0 - GAMMA
    en = (GAMMA - 2.0) / (GAMMA - 1.0) * a2
    rows, cols = [None] * 7, [None] * 7
    for i, o, z, x, y, G, w in ((0, 6, 1.0, af, as_, Gf, f), (2, 4, -1.0, as_, af, Gs, sl)):
        other = sl if z > 0 else f          # the fast pair couples to the slow speed and the other way round
        for j, e in ((i, 1.0), (o, -1.0)):
            rows[j] = [k * (-0.5 * g1 * x * u2 + e * G), k * (g1 * x * u[0] - e * x * w),
                       k * (g1 * x * u[1] + z * e * other * y * by * sg), k * (g1 * x * u[2] + z * e * other * y * bz * sg),
                       k * (g1 * x * b[1] + z * sr * c * y * by), k * (g1 * x * b[2] + z * sr * c * y * bz), -k * g1 * x]
            cols[j] = [x, x * (u[0] - e * w), x * u[1] + z * e * other * y * by * sg, x * u[2] + z * e * other * y * bz * sg,
                       z * c * y * by / sr, z * c * y * bz / sr, x * (0.5 * u2 + w * w - en) - e * G]
    for j, e in ((1, 1.0), (5, -1.0)):
        rows[j] = [0.5 * Ga, None, -0.5 * bz * sg, 0.5 * by * sg, -0.5 * e * sr * bz, 0.5 * e * sr * by, None]
        cols[j] = [None, None, -bz * sg, by * sg, -e * bz / sr, e * by / sr, -Ga]
    tau = -g1 / a2
    rows[3] = [1.0 - 0.5 * tau * u2, tau * u[0], tau * u[1], tau * u[2], tau * b[1], tau * b[2], -tau]
    cols[3] = [torch.ones_like(r), u[0], u[1], u[2], None, None, 0.5 * u2]
    out = [(7.0 * (x + _at(x, 1, axis)) - (_at(x, -1, axis) + _at(x, 2, axis))) / 12.0 for x in F]
    for j in range(7):
        a, b_ = [], []
        for o in range(-2, 3):              # the interfaces i-3/2 .. i+5/2
            sF = sum(rows[j][l] * _at(dF[l], o, axis) for l in range(7) if rows[j][l] is not None)
            sq = alpha[j] * sum(rows[j][l] * _at(dq[l], o, axis) for l in range(7) if rows[j][l] is not None)
            a.append(0.5 * (sF + sq))
            b_.append(0.5 * (sF - sq))
        d = _phi(b_[4], b_[3], b_[2], b_[1], weights) - _phi(a[0], a[1], a[2], a[3], weights)
        out = [x if cols[j][l] is None else x + cols[j][l] * d for l, x in enumerate(out)]
    mean = lambda x: 0.5 * (x + _at(x, 1, axis))
    return out[0], out[1], out[2], out[3], out[6], out[4] + mean(B[0] * v[1]), out[5] + mean(B[0] * v[2])


def _rhs(U, case, grad=False):
    walls, sizes = _walls(case), [case["nx"], case["ny"], case["nz"]]
    for a in walls:
        U = _double(U, a)
    rho, m, E, b = U
    ih = 1.0 / _h(case)
    B = _zone_b(b)
    P = _pressure(U, B)
    v = [x / rho for x in m]
    k, T = [0.0] * 5, {}
    for axis in range(3):
        flat = (rho, *m, E, *v, *B, P)
        fn = lambda *x, axis=axis: _sweep(axis, case["weights"], x[0], x[1:4], x[4], x[5:8], x[8:11], x[11])
        f = checkpoint(fn, *flat, use_reentrant=False) if grad else fn(*flat)
        t, s = (axis + 1) % 3, (axis + 2) % 3
        for o, c in ((0, 0), (1, 1 + axis), (2, 1 + t), (3, 1 + s), (4, 4)):
            k[c] = k[c] - (f[o] - _at(f[o], -1, axis)) * ih
        T[axis, t], T[axis, s] = f[5], f[6]
    avg = lambda x, a: 0.5 * (x + _at(x, 1, a))
    edge = [avg(T[2, 1], 1) - avg(T[1, 2], 2), avg(T[0, 2], 2) - avg(T[2, 0], 0), avg(T[1, 0], 0) - avg(T[0, 1], 1)]
    for a in walls:                         # no tangential electric field on a wall
        keep = torch.ones(2 * sizes[a], device=DEV, dtype=torch.float64)
        keep[[sizes[a] - 1, 2 * sizes[a] - 1]] = 0.0
        keep = keep.reshape([-1 if d == 2 - a else 1 for d in range(3)])
        edge = [e if c == a else e * keep for c, e in enumerate(edge)]
    diff = lambda x, a: (x - _at(x, -1, a)) * ih
    kb = [diff(edge[(c + 1) % 3], (c + 2) % 3) - diff(edge[(c + 2) % 3], (c + 1) % 3) for c in range(3)]
    for a in walls:
        k = [x.narrow(2 - a, 0, sizes[a]) for x in k]
        kb = [x.narrow(2 - a, 0, sizes[a]) for x in kb]
    return k[0], k[1:4], k[4], kb


def _add(U, k, c):
    return (U[0] + c * k[0], [x + c * y for x, y in zip(U[1], k[1])], U[2] + c * k[2],
            [x + c * y for x, y in zip(U[3], k[3])])


def _floored(U, case):
    if not case["floors"]:
        return U
    rho, m, E, b = U
    U = (rho.clamp(min=RHO_FLOOR), m, E, b)
    P = _pressure(U, _zone_b_walls(b, _walls(case)))
    return U[0], m, E + (P_FLOOR - P).clamp(min=0.0) / (GAMMA - 1.0), b


def _dt(U, case):
    rho, m, _, b = U
    B = _zone_b_walls(b, _walls(case))
    P = _pressure(U, B)
    top = [((m[a] / rho).abs() + _speeds(rho, B[a], (B[(a + 1) % 3], B[(a + 2) % 3]), P)[0]).max() for a in range(3)]
    return float(CFL[case["integrator"]] * _h(case) / (top[0] + top[1] + top[2]))


def _step(U, case, dt, grad=False):
    k0 = _rhs(U, case, grad)
    if case["integrator"] == "rk4":
        k1 = _rhs(_add(U, k0, 0.5 * dt), case, grad)
        k2 = _rhs(_add(U, k1, 0.5 * dt), case, grad)
        k3 = _rhs(_add(U, k2, dt), case, grad)
        return _add(_add(U, _add(k0, k3, 1.0), dt / 6.0), _add(k1, k2, 1.0), dt / 3.0)
    k1 = _rhs(_floored(_add(U, k0, dt), case), case, grad)
    U2 = _floored(_add(_add(U, k0, 0.25 * dt), k1, 0.25 * dt), case)
    k2 = _rhs(U2, case, grad)
    return _floored(_add(_add(_add(U, k0, dt / 6.0), k1, dt / 6.0), k2, 2.0 * dt / 3.0), case)


def _initial(case, rho, v, A):
    ih, back = 1.0 / _h(case), _background(case)
    d = lambda x, a: (x - _at(x, -1, a)) * ih
    b = [back[c] + (d(A[(c + 2) % 3], (c + 1) % 3) - d(A[(c + 1) % 3], (c + 2) % 3)) for c in range(3)]
    for a in _walls(case):
        b[a] = b[a].clone()
        b[a].select(2 - a, b[a].shape[2 - a] - 1).zero_()
    round_ = (lambda x: x.float().double()) if case["precision"] == "fp32" else (lambda x: x)
    b = [round_(x) for x in b]
    B = [round_(x) for x in _zone_b_walls(b, _walls(case))]
    m = [rho * v[c] for c in range(3)]
    E = P0 / (GAMMA - 1.0) + 0.5 * (sum(m[c] * v[c] for c in range(3)) + sum(x * x for x in B))
    return round_(rho), [round_(x) for x in m], round_(E), b


def _hydro(U):
    return torch.stack([U[0], *U[1], U[2]])


def exact(case, seed):
    path = case["path"]
    if case["nx"] * case["ny"] * case["nz"] > 3e7:
        return None                         # over about 20 seconds
    rho, v, A = _fields(case, seed)
    if path == "gradient":
        A, v = A.requires_grad_(), v.requires_grad_()
        U = _initial(case, rho, v, A)
        for _ in range(case["steps"]):
            with torch.no_grad():
                dt = _dt(U, case)
            U = _step(U, case, dt, grad=True)
        out = _hydro(U), torch.stack(U[3])
        gA, gv = torch.autograd.grad(out, (A, v), _cotangents(case, seed))
        return out[0].detach(), out[1].detach(), gA, gv
    U = _initial(case, rho, v, A)
    if path == "adjoint":
        x = [_hydro(U).requires_grad_(), torch.stack(U[3]).requires_grad_()]
        dt = _dt(U, case)
        U = _step((x[0][0], list(x[0][1:4]), x[0][4], list(x[1])), case, dt, grad=True)
        return torch.autograd.grad((_hydro(U), torch.stack(U[3])), x, _cotangents(case, seed))
    if path == "monitor":
        B = _zone_b_walls(U[3], _walls(case))
        P = _pressure(U, B)
        total = lambda x: float(x.sum())
        # the divergence is rounding alone: no value in 64 bits
        return dict(max_divb=None, mass=total(U[0]), mom=[total(x) for x in U[1]], energy=total(U[2]),
                    bflux=[total(x) for x in U[3]], min_rho=float(U[0].min()), min_p=float(P.min()),
                    n_unphysical=int(((P <= 0) | (U[0] <= 0)).sum()), n_floored=0, dt=_dt(U, case))
    for _ in range(GRAPH_STEPS if path == "graph" else 1):
        U = _step(U, case, _dt(U, case))
    return _hydro(U), torch.stack(U[3]), torch.stack(_zone_b_walls(U[3], _walls(case)))
