"""Workloads of the GRMHD library as its users call it, for timing and for comparing results.

A case is a dict of plain values.  ``prepare`` makes what a program holds before the call (seeded
inputs on the GPU and a solver), ``run`` makes one pass through the public entry points, ``work``
counts what a pass cannot do without, and ``exact`` evaluates the same discretisation in plain
float64 torch, without the library.  Kinds of pass:

  evolve    primitives -> conserved variables, a stretch of Runge-Kutta steps, -> primitives
  rhs       one right-hand side (the caller integrates in time itself)
  gradient  a differentiable evolution, forward and backward
  ensemble  many uneven 1D problems advanced together
"""
import math
import random

import torch

from paper_1102_5202_amd import adjoint, grmhd

DEV = "cuda:0"
GAMMA = {"box": 4.0 / 3.0, "blob": 2.0, "tube": 5.0 / 3.0}
HALF = 20.0          # the blob's box is [-HALF, HALF]^3
K_POLY = 100.0


def _grid(kind, data, n, steps, **over):
    c = {"kind": kind, "data": data, "nx": n[0], "ny": n[1], "nz": n[2], "steps": steps,
         "metric": "iso" if data == "blob" else "flat", "precision": "fp64",
         "rk": 2 if data == "box" else 3, "recon": "mc", "div": "cleaning"}
    c.update(over)
    return c


def listed():
    return [
        # one right-hand side of a small block inside somebody else's time integrator: launches
        # and latency only
        {"name": "rhs_24x20x16", **_grid("rhs", "blob", (24, 20, 16), 1)},
        # the 1D shock-tube problems of every code test: 400 cells, a stretch of its 400 steps
        {"name": "tube_400", **_grid("evolve", "tube", (400, 1, 1), 20)},
        # a 2D run of ordinary size
        {"name": "plane_500x300", **_grid("evolve", "box", (500, 300, 1), 5, rk=3)},
        # the periodic box at the size of the inverse problems, forward only
        {"name": "box_64", **_grid("evolve", "box", (64, 64, 64), 5)},
        # the periodic box at its full size in the mixed precision of production runs
        {"name": "box_128_mixed", **_grid("evolve", "box", (128, 128, 128), 5, precision="mixed")},
        # an odd-sized block of the curved workload, as a domain decomposition leaves it
        {"name": "blob_101x87x75", **_grid("evolve", "blob", (101, 87, 75), 3)},
        # the benchmark workload: the curved blob at 192^3, FP64
        {"name": "blob_192", **_grid("evolve", "blob", (192, 192, 192), 3)},
        # the scheme's options: parabolic reconstruction, flux-CT, a spacetime given on the grid
        {"name": "blob_ppm_128", **_grid("evolve", "blob", (128, 128, 128), 2, recon="ppm")},
        {"name": "box_fluxct_128", **_grid("evolve", "box", (128, 128, 128), 3, div="fluxct")},
        {"name": "stored_96x80x72", **_grid("evolve", "blob", (96, 80, 72), 3, metric="stored")},
        # the inverse problem: the gradient through a stretch of steps of the periodic box
        {"name": "gradient_64", **_grid("gradient", "box", (64, 64, 64), 6, every=6)},
        # the batched ensemble of 256 uneven shock tubes, each to an early time with its own step
        {"name": "ensemble_256", "kind": "ensemble", "nprob": 256, "nmin": 200, "nmax": 4000, "t_end": 0.04,
         "precision": "fp64"},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("rhs", "tube", "plane", "grid", "grid", "grid", "option", "option", "gradient", "ensemble"))
    if kind == "rhs":
        return _grid("rhs", rng.choice(("box", "blob")), tuple(size(10, 44) for _ in range(3)), 1)
    if kind == "tube":
        return _grid("evolve", "tube", (size(50, 8192), 1, 1), rng.randint(5, 30),
                     precision=rng.choice(("fp64", "fp64", "mixed")))
    if kind == "plane":
        return _grid("evolve", "box", (size(32, 1024), size(32, 1024), 1), rng.randint(2, 6),
                     rk=rng.choice((2, 3)), precision=rng.choice(("fp64", "fp64", "mixed")))
    if kind == "gradient":
        steps = rng.randint(2, 6)
        return _grid("gradient", "box", tuple(size(16, 64) for _ in range(3)), steps,
                     every=rng.choice((steps, (steps + 1) // 2)))
    if kind == "ensemble":
        nmin = size(50, 1000)
        return {"kind": "ensemble", "nprob": size(8, 200), "nmin": nmin, "nmax": size(nmin, 4000),
                "t_end": round(rng.uniform(0.01, 0.04), 3), "precision": rng.choice(("fp64", "mixed"))}
    n = tuple(size(16, 192) for _ in range(3))
    data = rng.choice(("box", "blob"))
    if kind == "grid":
        return _grid("evolve", data, n, rng.randint(1, 3), precision=rng.choice(("fp64", "fp64", "mixed")))
    over = rng.choice(({"recon": "ppm"}, {"div": "fluxct"}, {"metric": "stored"}))
    n = tuple(min(v, 128) for v in n)
    return _grid("evolve", "blob" if "metric" in over else data, n, rng.randint(1, 2), **over)


# ------------------------------------------------------------------------------------------------
# inputs

def _box_of(case):
    n = (case["nx"], case["ny"], case["nz"])
    if case["data"] == "blob":
        return n, (-HALF,) * 3, (HALF,) * 3, (grmhd.OUTFLOW,) * 3
    bc = grmhd.PERIODIC if case["data"] == "box" else grmhd.OUTFLOW
    return n, (0.0,) * 3, (1.0,) * 3, (bc,) * 3


def _dt(case):
    """Courant number 0.4 of an unsplit update, signal speeds at most 1."""
    n, lo, hi, _ = _box_of(case)
    return 0.4 / sum(n[a] / (hi[a] - lo[a]) for a in range(3) if n[a] > 1)


def _floors(case):
    return (1e-10, K_POLY * 1e-20) if case["data"] == "blob" else (1e-12, 1e-12)


def _coords(case, shift=(0.0, 0.0, 0.0), ghost=0):
    n, lo, hi, _ = _box_of(case)
    xs = []
    for a in range(3):
        g = ghost if n[a] > 1 else 0
        i = torch.arange(-g, n[a] + g, dtype=torch.float64, device=DEV)
        xs.append(lo[a] + (i + 0.5 + shift[a]) * ((hi[a] - lo[a]) / n[a]))
    return xs[0][None, None, :], xs[1][None, :, None], xs[2][:, None, None]


def _uniform(gen, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV)


def _tube_states(gen):
    """Left and right states of a magnetised Riemann problem."""
    r = _uniform(gen, 0.0, 1.0, 9)
    z = torch.zeros((), dtype=torch.float64, device=DEV)
    bx = 0.3 + 0.7 * r[4]
    sides = [torch.stack([0.1 + 0.9 * r[s], 0.01 + 0.99 * r[2 + s], z, z, z, bx, 2.0 * r[5 + 2 * s] - 1.0,
                          2.0 * r[6 + 2 * s] - 1.0, z]) for s in (0, 1)]
    return sides


def _tube(gen, n):
    left, right = _tube_states(gen)
    x = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
    return torch.where(x < 0.5, left[:, None], right[:, None])


def _box(case, gen):
    """Smooth flow in a periodic box: Fourier modes in density, pressure, velocity and field (the
    field's modes transverse to their wave vectors) on a uniform background field."""
    n = (case["nx"], case["ny"], case["nz"])
    X = _coords(case)
    shape = (n[2], n[1], n[0])
    modes = 8
    act = torch.tensor([1.0 if n[a] > 1 else 0.0 for a in range(3)], dtype=torch.float64, device=DEV)

    def draw_modes():
        k = torch.round(_uniform(gen, -3.0, 3.0, modes, 3)) * act
        k[:, 0] += (k.abs().sum(dim=1) == 0)
        return k, _uniform(gen, 0.0, 2 * math.pi, modes), _uniform(gen, -1.0, 1.0, modes)

    def phase(k, ph, m):
        return 2 * math.pi * (k[m, 0] * X[0] + k[m, 1] * X[1] + k[m, 2] * X[2]) + ph[m]

    def scalar():
        k, ph, am = draw_modes()
        f = torch.zeros(shape, dtype=torch.float64, device=DEV)
        for m in range(modes):
            f += (am[m] / am.abs().sum()) * torch.cos(phase(k, ph, m))
        return f

    P = torch.zeros((9,) + shape, dtype=torch.float64, device=DEV)
    P[0] = 1.0 + 0.1 * scalar()
    P[1] = 0.1 * (1.0 + 0.05 * scalar())
    v = [0.3 / math.sqrt(3.0) * scalar() for _ in range(3)]
    W = torch.rsqrt(1.0 - (v[0] ** 2 + v[1] ** 2 + v[2] ** 2))
    for i in range(3):
        P[2 + i] = W * v[i]
    k, ph, am = draw_modes()
    pol = torch.linalg.cross(k, _uniform(gen, -1.0, 1.0, modes, 3))
    pol = 0.01 * pol / pol.norm(dim=1).sum()
    for i, b0 in enumerate((0.1, 0.05, 0.0)):
        P[5 + i] = b0
        for m in range(modes):
            P[5 + i] += pol[m, i] * torch.cos(phase(k, ph, m))
    if case["kind"] == "gradient":
        # a cleaning scalar away from zero: a uniform one sits on the limiter's kink, where the
        # step has no derivative
        P[8] = 1e-3 * scalar()
    return P


def _blob(case, gen):
    """A rotating, magnetised polytropic blob around the origin with an atmosphere."""
    n = (case["nx"], case["ny"], case["nz"])
    X = _coords(case)
    shape = (n[2], n[1], n[0])
    r2 = X[0] ** 2 + X[1] ** 2 + X[2] ** 2
    P = torch.zeros((9,) + shape, dtype=torch.float64, device=DEV)
    rho_atm, _ = _floors(case)
    P[0] = torch.clamp(1e-3 * torch.exp(-r2 / 16.0) * (1.0 + 0.01 * _uniform(gen, -1.0, 1.0, *shape)), min=rho_atm)
    P[1] = K_POLY * P[0] ** 2
    alpha, psi4 = _isotropic(r2)
    omega = 0.02
    vx, vy = -omega * X[1] / alpha, omega * X[0] / alpha
    W = torch.rsqrt(1.0 - psi4 * (vx ** 2 + vy ** 2))
    P[2] = W * vx
    P[3] = W * vy

    # the densitised field as the central curl of (-y, x, 0) times the envelope
    dx = [2 * HALF / v for v in n]

    def A(axis, s):
        Y = _coords(case, shift=s)
        env = torch.exp(-(Y[0] ** 2 + Y[1] ** 2 + Y[2] ** 2) / 16.0)
        return (-Y[1] if axis == 0 else Y[0]) * env

    def d(axis, along):
        e = [0.0, 0.0, 0.0]
        e[along] = 1.0
        return (A(axis, e) - A(axis, [-v for v in e])) / (2 * dx[along])

    B = torch.stack([-d(1, 2), d(0, 2), d(1, 0) - d(0, 1)]) / (alpha * psi4 ** 1.5)
    b2 = psi4 * (B * B).sum(dim=0)
    P[5:8] = B * torch.sqrt((P[1].max() / 1000.0) / (0.5 * b2.max()))
    return P


def _isotropic(r2):
    """Lapse and psi^4 of the isotropic Schwarzschild metric, M = 1, r_s = sqrt(r^2 + 1)."""
    h = 0.5 / torch.sqrt(r2 + 1.0)
    return (1.0 - h) / (1.0 + h), (1.0 + h) ** 4


def _stored_metric(case):
    X = _coords(case, ghost=2)
    return [m.contiguous() for m in _isotropic(X[0] ** 2 + X[1] ** 2 + X[2] ** 2)]


def _lengths(case):
    """Cells and steps (dt = 0.4 / n to t_end) of each problem: the ensemble's own, whatever the seed."""
    rng = random.Random(case["nprob"] * 100003 + case["nmin"] * 317 + case["nmax"])
    n = [rng.randint(case["nmin"], case["nmax"]) for _ in range(case["nprob"])]
    return n, [max(1, round(case["t_end"] * v / 0.4)) for v in n]


def _inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    if case["kind"] == "ensemble":
        return [_tube(gen, v) for v in _lengths(case)[0]]
    if case["data"] == "tube":
        return _tube(gen, case["nx"]).reshape(9, 1, 1, case["nx"]).contiguous()
    return _box(case, gen) if case["data"] == "box" else _blob(case, gen)


def _options(case):
    n, lo, hi, bc = _box_of(case)
    rho_atm, p_atm = _floors(case)
    metric = {"flat": grmhd.FLAT, "iso": grmhd.ISO_SCHW, "stored": grmhd.STORED}[case["metric"]]
    return dict(n=n, lo=lo, hi=hi, bc=bc, metric=metric, M=1.0 if case["metric"] == "iso" else 0.0, r_min=1.0,
                gamma=GAMMA[case["data"]], rk_order=case["rk"], rho_atm=rho_atm, p_atm=p_atm,
                precision=case["precision"], reconstruction=case["recon"], divergence=case["div"])


# ------------------------------------------------------------------------------------------------
# the passes

def prepare(case, seed):
    st = {"case": case}
    if case["kind"] == "ensemble":
        n, steps = _lengths(case)
        st["solver"] = s = grmhd.BatchSolver(n, [0.0] * len(n), [1.0] * len(n), [0.4 / v for v in n], steps,
                                             precision=case["precision"], device=DEV)
        st["P"], st["U"], st["Pout"] = s.pack(_inputs(case, seed)), s.empty(), s.empty()
        s.cons(st["P"], st["U"])
        s.tune(st["U"], 10)     # once per ensemble, before the run
        return st
    st["P"] = _inputs(case, seed)
    opts = _options(case)
    if case["kind"] == "rhs":
        st["R"] = torch.empty_like(st["P"])
        st["opts"] = opts
        return st
    if case["kind"] == "gradient":
        st["P"].requires_grad_(True)
        st["solver"] = grmhd.Solver(adjoint=True, tape_steps=case["every"], device=DEV, **opts)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(int(seed) + 1)
        st["Pbar"] = _uniform(gen, -1.0, 1.0, *st["P"].shape)
        return st
    st["solver"] = s = grmhd.Solver(device=DEV, **opts)
    if case["metric"] == "stored":
        s.set_metric(*_stored_metric(case))
    st["U"], st["Pout"] = s.empty(), s.empty()
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "rhs":
        return grmhd.rhs_noalloc(state["P"], R=state["R"], **state["opts"])
    s = state["solver"]
    if case["kind"] == "gradient":
        P = adjoint.evolve(s, state["P"], _dt(case), case["steps"], case["every"])
        (g,) = torch.autograd.grad(P, state["P"], state["Pbar"])
        return {"P": P.detach(), "grad": g}
    U = s.cons(state["P"], state["U"])
    if case["kind"] == "ensemble":
        s.evolve(U)
    else:
        dt = _dt(case)
        for _ in range(case["steps"]):
            s.step(U, dt)
    P = s.prim(U, state["Pout"])
    return {"U": U, "P": P}


def work(case):
    """Bytes: a grid's substep reads the primitives and U^n and writes both new ones (its stencil
    spans the grid, so they pass through memory; mixed precision holds the primitives and the stage
    state in 4 bytes); the conversions read one array and write one.  An ensemble's problem can stay
    on its compute unit: read and written once.  Operations: about 500 for a face (reconstruction,
    two states, fluxes), 400 for a cell (recovery, combination)."""
    if case["kind"] == "ensemble":
        n, steps = _lengths(case)
        return {"bytes": sum(n) * 8 * 9 * 4, "flops": sum(v * k for v, k in zip(n, steps)) * 3 * 900.0}
    N = case["nx"] * case["ny"] * case["nz"]
    faces = sum(1 for a in ("nx", "ny", "nz") if case[a] > 1) * 500.0
    if case["kind"] == "rhs":
        return {"bytes": N * 8 * 18, "flops": N * (faces + 100.0)}
    sub = case["steps"] * case["rk"]
    per = 288.0 if case["precision"] == "fp64" else 216.0
    bytes_, flops = N * (per * sub + 8 * 36), N * ((faces + 400.0) * sub + 300.0)
    if case["kind"] == "gradient":
        # back: the stage's primitives and the cotangents of U, U^n and R read, the last three written
        return {"bytes": 2 * bytes_ + N * sub * 72.0 * 7, "flops": flops * 4}
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------------------------------------------
# the same discretisation in plain float64 torch

class _Plain:
    """One grid (or, with ``segments``, many 1D rows side by side): each axis' ghosted positions,
    and for every cell the faces on its two sides along that axis."""

    def __init__(self, case, segments=None, dx=None):
        self.case, self.segments = case, segments
        if segments is not None:
            self.axes, self.bc, self.dx = [0], [1, 1, 1], [dx, None, None]
            self.gamma, self.rk, self.recon, self.ct = GAMMA["tube"], 3, "mc", False
            self.rho_atm, self.p_atm, self.metric = 1e-12, 1e-12, "flat"
        else:
            self.n, lo, hi, self.bc = _box_of(case)
            self.dx = [(hi[a] - lo[a]) / self.n[a] for a in range(3)]
            self.axes = [a for a in range(3) if self.n[a] > 1]
            self.gamma, self.rk = GAMMA[case["data"]], case["rk"]
            self.recon, self.ct = case["recon"], case["div"] == "fluxct"
            self.rho_atm, self.p_atm = _floors(case)
            self.metric = case["metric"]
        self.g = 3 if self.recon == "ppm" else 2
        self.ghosted, self.left = {}, {}
        for a in self.axes:
            idx, left, at = [], [], 0
            for n in (segments if segments is not None else [self.n[a]]):
                j = torch.arange(-self.g, n + self.g, device=DEV)
                idx.append((j % n if self.bc[a] == grmhd.PERIODIC else j.clamp(0, n - 1)) + at)
                left.append(torch.arange(n, device=DEV) + at + 2 * self.g * len(left))
                at += n
            self.ghosted[a], self.left[a] = torch.cat(idx), torch.cat(left)
        self.geo_c, self.dalpha, self.dpsi4 = self._centre_geometry()
        self.geo_f = {a: self._face_geometry(a) for a in self.axes}

    # geometry: (alpha, psi^4, sqrt(gamma), sqrt(-g))
    @staticmethod
    def _geo(alpha, psi4):
        sg = psi4 ** 1.5
        return alpha, psi4, sg, alpha * sg

    def _centre_geometry(self):
        one = torch.ones((), dtype=torch.float64, device=DEV)
        if self.metric == "flat":
            return self._geo(one, one), None, None
        if self.metric == "stored":
            self.stored = _stored_metric(self.case)
            inner = [self._inner(m, ()) for m in self.stored]
            d = []
            for m in self.stored:
                row = []
                for a in range(3):
                    if a not in self.axes:
                        row.append(torch.zeros_like(inner[0]))
                        continue
                    x, dim, n = self._inner(m, (a,)), 2 - a, self.n[a]
                    t = [x.narrow(dim, o, n) for o in (0, 1, 3, 4)]
                    row.append((t[0] - 8 * t[1] + 8 * t[2] - t[3]) / (12 * self.dx[a]))
                d.append(row)
            return self._geo(*inner), d[0], d[1]
        X = _coords(self.case)
        r2 = X[0] ** 2 + X[1] ** 2 + X[2] ** 2
        alpha, psi4 = _isotropic(r2)
        rs = torch.sqrt(r2 + 1.0)
        h = 0.5 / rs
        ka, kp = 2 * h / (rs ** 2 * (1 + h) ** 2), -4 * (1 + h) ** 3 * h / rs ** 2
        return self._geo(alpha, psi4), [ka * X[a] for a in range(3)], [kp * X[a] for a in range(3)]

    def _inner(self, m, keep):
        """The interior of a ghosted metric array along the axes not in ``keep``."""
        for a in range(3):
            if a not in keep and self.n[a] > 1:
                m = m.narrow(2 - a, 2, self.n[a])
        return m

    def _face_geometry(self, a):
        if self.metric == "flat":
            return self.geo_c
        n = self.n[a]
        if self.metric == "stored":
            out = []
            for m in self.stored:
                x = self._inner(m, (a,))
                t = [x.narrow(2 - a, o, n + 1) for o in range(4)]
                out.append((-t[0] + 9 * t[1] + 9 * t[2] - t[3]) / 16.0)
            return self._geo(*out)
        X = list(_coords(self.case))
        shape = [1, 1, 1]
        shape[2 - a] = n + 1
        X[a] = (-HALF + torch.arange(n + 1, dtype=torch.float64, device=DEV) * self.dx[a]).reshape(shape)
        return self._geo(*_isotropic(X[0] ** 2 + X[1] ** 2 + X[2] ** 2))

    # point physics
    def kinematics(self, q, geo):
        alpha, psi4 = geo[0], geo[1]
        rho, p, u, B = q[0], q[1], q[2:5], q[5:8]
        W = torch.sqrt(1 + psi4 * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2))
        ut = W / alpha
        bt = psi4 * (B[0] * u[0] + B[1] * u[1] + B[2] * u[2])
        b = [(B[i] + bt * u[i]) / ut for i in range(3)]
        b2 = (psi4 * (B[0] ** 2 + B[1] ** 2 + B[2] ** 2) + bt ** 2) / ut ** 2
        w = rho + self.gamma / (self.gamma - 1) * p
        return W, bt, b, b2, w

    def conserved(self, q, geo):
        alpha, psi4, sg, smg = geo
        W, bt, b, b2, w = self.kinematics(q, geo)
        wt, pt = w + b2, q[1] + 0.5 * b2
        D = sg * q[0] * W
        tau = smg * (wt * W ** 2 - pt - (alpha * bt) ** 2) - D
        S = [psi4 * (sg * wt * W * q[2 + j] - smg * bt * b[j]) for j in range(3)]
        return torch.stack([D, tau, *S, smg * q[5], smg * q[6], smg * q[7], q[8]])

    def flux(self, q, geo, a):
        alpha, psi4, sg, smg = geo
        W, bt, b, b2, w = self.kinematics(q, geo)
        wt, pt, u = w + b2, q[1] + 0.5 * b2, q[2:5]
        F = [smg * q[0] * u[a], smg * ((wt * alpha * W - q[0]) * u[a] - alpha ** 2 * bt * b[a])]
        F += [smg * (psi4 * (wt * u[a] * u[j] - b[a] * b[j]) + (pt if j == a else 0.0)) for j in range(3)]
        F += [smg * (b[j] * u[a] - b[a] * u[j]) for j in range(3)]
        c2 = (self.gamma * q[1] + b2) / wt
        den = W ** 2 * (1 - c2) + c2
        root = torch.sqrt(torch.clamp(c2 * (den / psi4 - u[a] ** 2 * (1 - c2)), min=0.0))
        return F, alpha * (W * u[a] * (1 - c2) - root) / den, alpha * (W * u[a] * (1 - c2) + root) / den

    @staticmethod
    def slope(m, c, p):
        dl, dr, dc = c - m, p - c, 0.5 * (p - m)
        s = torch.sign(dc) * torch.minimum(torch.minimum(2 * dl.abs(), 2 * dr.abs()), dc.abs())
        return torch.where(dl * dr > 0, s, torch.zeros_like(s))

    def edges(self, Pg, dim):
        """Left and right edge values of every ghosted cell that has its stencil."""
        def at(x, o, cut):
            return x.narrow(dim, o, x.shape[dim] - cut)
        s = self.slope(at(Pg, 0, 2), at(Pg, 1, 2), at(Pg, 2, 2))
        if self.recon == "mc":
            c = at(Pg, 1, 2)
            return c - 0.5 * s, c + 0.5 * s
        c, m, p = at(Pg, 2, 4), at(Pg, 1, 4), at(Pg, 3, 4)
        sm, s0, sp = at(s, 0, 2), at(s, 1, 2), at(s, 2, 2)
        lo = 0.5 * (m + c) - (s0 - sm) / 6
        hi = 0.5 * (c + p) - (sp - s0) / 6
        flat = (hi - c) * (c - lo) <= 0
        d, m6 = hi - lo, 6 * (c - 0.5 * (lo + hi))
        lo2 = torch.where(d * m6 > d * d, 3 * c - 2 * hi, lo)
        hi2 = torch.where(-d * d > d * m6, 3 * c - 2 * lo, hi)
        return torch.where(flat, c, lo2), torch.where(flat, c, hi2)

    def faces(self, P, a):
        dim = P.dim() - 1 - a
        eL, eR = self.edges(P.index_select(dim, self.ghosted[a]), dim)
        # face between consecutive cells: the right edge below it, the left edge above it
        m = eL.shape[dim] - 1
        qL, qR, geo = eR.narrow(dim, 0, m), eL.narrow(dim, 1, m), self.geo_f[a]
        smg = geo[3]
        BL, BR = smg * qL[5 + a], smg * qR[5 + a]
        if self.ct:
            Bs = 0.5 * (BL + BR)
        else:
            Bs, phs = 0.5 * (BL + BR) - 0.5 * (qR[8] - qL[8]), 0.5 * (qL[8] + qR[8]) - 0.5 * (BR - BL)
        qL, qR = list(qL.unbind(0)), list(qR.unbind(0))
        qL[5 + a] = qR[5 + a] = Bs / smg
        FL, mL, pL = self.flux(qL, geo, a)
        FR, mR, pR = self.flux(qR, geo, a)
        UL, UR = self.conserved(qL, geo), self.conserved(qR, geo)
        sl = torch.clamp(torch.minimum(mL, mR), max=0.0)
        sr = torch.clamp(torch.maximum(pL, pR), min=0.0)
        F = [(sr * FL[v] - sl * FR[v] + sl * sr * (UR[v] - UL[v])) / (sr - sl) for v in range(8)]
        F[5 + a] = torch.zeros_like(Bs) if self.ct else phs
        F.append(torch.zeros_like(Bs) if self.ct else Bs)
        return torch.stack(F)

    def constrained(self, F):
        """Flux-CT: transverse field fluxes from the edge averages of the face fluxes."""
        out = {a: F[a].clone() for a in self.axes}
        for a in self.axes:
            for b in self.axes:
                if a >= b:
                    continue
                def both(x, axis):
                    dim, n = x.dim() - 1 - axis, self.n[axis]
                    j = torch.arange(-1, n + 1, device=DEV)
                    j = j % n if self.bc[axis] == grmhd.PERIODIC else j.clamp(0, n - 1)
                    return x.index_select(dim, j[:-1]) + x.index_select(dim, j[1:])
                E = 0.25 * (both(F[b][5 + a], a) - both(F[a][5 + b], b))

                def mean(x, axis):
                    dim, n = x.dim() - 1 - axis, self.n[axis]
                    return 0.5 * (x.narrow(dim, 0, n) + x.narrow(dim, 1, n))
                out[a][5 + b] = -mean(E, b)
                out[b][5 + a] = mean(E, a)
        # two pairs never write the same component: (a, 5 + b) belongs to the pair {a, b} alone
        return out

    def rhs(self, P):
        F = {a: self.faces(P, a) for a in self.axes}
        if self.ct and len(self.axes) > 1:
            F = self.constrained(F)
        R = 0.0
        for a in self.axes:
            dim = P.dim() - 1 - a
            R = R - (F[a].index_select(dim, self.left[a] + 1) - F[a].index_select(dim, self.left[a])) / self.dx[a]
        R = list(R.unbind(0))
        if self.dalpha is not None:
            alpha, psi4, sg, smg = self.geo_c
            W, bt, b, b2, w = self.kinematics(P, self.geo_c)
            wt, pt = w + b2, P[1] + 0.5 * b2
            Ttt = (wt * W ** 2 - pt) / alpha ** 2 - bt ** 2
            Tkk = wt * (P[2] ** 2 + P[3] ** 2 + P[4] ** 2) + 3 * pt / psi4 - (b[0] ** 2 + b[1] ** 2 + b[2] ** 2)
            for j in range(3):
                R[2 + j] = R[2 + j] + smg * (0.5 * Tkk * self.dpsi4[j] - alpha * Ttt * self.dalpha[j])
        if not self.ct:
            R[8] = R[8] - P[8]
        return torch.stack(R)

    # recovery: Newton on the energy equation in Wc = rho h W^2 with v^2 eliminated
    def _residual(self, Wc, D, E, Q2, B2, QB2):
        s = B2 + Wc
        v2 = (Q2 + QB2 * (B2 + 2 * Wc) / Wc ** 2) / s ** 2
        dv2 = -2 * (Q2 + QB2 * (3 * Wc * s + B2 ** 2) / Wc ** 3) / s ** 3
        gk = (self.gamma - 1) / self.gamma
        root = torch.sqrt(torch.clamp(1 - v2, min=1e-300))
        p = gk * (Wc * (1 - v2) - D * root)
        f = E - Wc + p - 0.5 * B2 * (1 + v2) + 0.5 * QB2 / Wc ** 2
        df = -1 + gk * (1 - v2 + (0.5 * D / root - Wc) * dv2) - 0.5 * B2 * dv2 - QB2 / Wc ** 3
        return f, df, v2, p

    def primitives(self, U, guess):
        alpha, psi4, sg, smg = self.geo_c
        D, E = U[0] / sg, (U[1] + U[0]) / smg
        Q, B = [U[2 + i] / sg for i in range(3)], [U[5 + i] / sg for i in range(3)]
        Q2 = (Q[0] ** 2 + Q[1] ** 2 + Q[2] ** 2) / psi4
        B2 = psi4 * (B[0] ** 2 + B[1] ** 2 + B[2] ** 2)
        QB = Q[0] * B[0] + Q[1] * B[1] + Q[2] * B[2]
        with torch.no_grad():
            args = [x.detach() for x in (D, E, Q2, B2, QB ** 2)]
            W2 = 1 + psi4 * (guess[2] ** 2 + guess[3] ** 2 + guess[4] ** 2)
            Wc = ((guess[0] + self.gamma / (self.gamma - 1) * guess[1]) * W2).detach()
            last, more = torch.full_like(Wc, math.inf), 3
            for _ in range(60):
                f, df, v2, _p = self._residual(Wc, *args)
                new = torch.where(v2 < 1, Wc - f / df, 2 * Wc)
                new = torch.where(new > 0, new, 0.5 * Wc)
                step, Wc = ((new - Wc).abs() / new).max(), new
                more = more - 1 if float(step) < 1e-10 else 3
                if more == 0:
                    break
        f, df, _, _ = self._residual(Wc, D, E, Q2, B2, QB ** 2)
        Wc = Wc - f / df.detach()     # its derivative is the implicit function theorem's
        _, _, v2, p = self._residual(Wc, D, E, Q2, B2, QB ** 2)
        W = torch.rsqrt(1 - v2)
        u = [W * (Q[i] / psi4 + QB / Wc * B[i]) / (Wc + B2) for i in range(3)]
        rho = D / W
        atm = ~(rho >= (1 - 1e-10) * self.rho_atm)
        low = ~(torch.where(atm, torch.full_like(p, self.p_atm), p) >= self.p_atm)
        rho = torch.where(atm, torch.full_like(rho, self.rho_atm), rho)
        p = torch.where(atm | low, torch.full_like(p, self.p_atm), p)
        u = [torch.where(atm, torch.zeros_like(x), x) for x in u]
        P = torch.stack([rho, p, *u, U[5] / smg, U[6] / smg, U[7] / smg, U[8]])
        rebuilt = self.conserved(P, self.geo_c)
        return P, torch.cat([torch.where(atm | low, rebuilt[:5], U[:5]), U[5:]])

    def step(self, U, P, dt):
        stages = ((0.0, 1.0), (0.75, 0.25), (1 / 3, 2 / 3)) if self.rk == 3 else ((0.0, 1.0), (0.5, 0.5))
        Un = U
        for a, b in stages:
            P, U = self.primitives(U + a * (Un - U) + b * (dt * self.rhs(P)), P)
        return U, P


def exact(case, seed):
    if case["kind"] == "ensemble":
        (n, steps), rows = _lengths(case), _inputs(case, seed)
        seg = torch.cat([torch.full((v,), float(v), dtype=torch.float64, device=DEV) for v in n])
        left = torch.cat([torch.full((v,), k, device=DEV) for v, k in zip(n, steps)])
        s = _Plain(case, segments=n, dx=1.0 / seg)
        P = torch.cat(rows, dim=1)
        U, dt = s.conserved(P, s.geo_c), 0.4 / seg
        for k in range(max(steps)):
            U1, P1 = s.step(U, P, dt)
            on = left > k
            U, P = torch.where(on, U1, U), torch.where(on, P1, P)
        P, _ = s.primitives(U, P)
        return {"U": _packed(U, n), "P": _packed(P, n)}
    s = _Plain(case)
    P = _inputs(case, seed)
    if case["kind"] == "rhs":
        return s.rhs(P)
    if case["kind"] == "gradient":
        P0 = P.requires_grad_(True)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(int(seed) + 1)
        Pbar = _uniform(gen, -1.0, 1.0, *P0.shape)
        U, P = s.conserved(P0, s.geo_c), P0
        for _ in range(case["steps"]):
            U, P = s.step(U, P, _dt(case))
        P, _ = s.primitives(U, P)
        (g,) = torch.autograd.grad(P, P0, Pbar)
        return {"P": P.detach(), "grad": g}
    with torch.no_grad():
        U = s.conserved(P, s.geo_c)
        for _ in range(case["steps"]):
            U, P = s.step(U, P, _dt(case))
        P, _ = s.primitives(U, P)
    return {"U": U, "P": P}


def _packed(x, n):
    return torch.cat([part.reshape(-1) for part in x.split(n, dim=1)])
