"""The one-launch FP64 substep and right-hand side at the sizes where their split
can go wrong, against the oracle: rows shorter and longer than the 62 positions
of a wave, rows that end on its edges, one and several planes a wave, axes of
one, two and three cells, every combination of active axes, both boundary
rules.  Bars as for the other FP64 comparisons: 1e-11 of the largest value for a
right-hand side, 1e-10 relative L1 after steps."""
import numpy as np
import pytest
import torch

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SIZES = [(2, 1, 1), (61, 1, 1), (62, 1, 1), (63, 1, 1), (125, 1, 1), (1, 70, 1), (1, 1, 70), (60, 3, 1), (31, 2, 2),
         (1, 5, 70), (64, 1, 9), (2, 2, 2), (3, 3, 3), (62, 4, 5), (7, 37, 3), (190, 2, 17)]


@pytest.fixture(scope="module")
def G():
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    return grmhd


def _workload(n, bc, metric, seed):
    """Seeded rough data around a moving, magnetised state."""
    rng = np.random.default_rng(seed)
    base = np.array([1.0, 0.2, 0.2, -0.15, 0.1, 0.15, 0.1, -0.1, 0.02])
    P = base[:, None, None, None] * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (9, n[2], n[1], n[0])))
    lo, hi = ((2.0, 1.0, 1.5), (4.0, 3.0, 3.5)) if metric else ((0.0,) * 3, (1.0,) * 3)
    return WL.Workload(name="rough_%dx%dx%d" % n, P=P, n=n, lo=lo, hi=hi, bc=(bc,) * 3, gamma=4.0 / 3.0, rk_order=3,
                       dt=0.5 * WL.cfl_dt(n, lo, hi), nsteps=2, metric=WL.ISO_SCHW if metric else WL.FLAT,
                       M=1.0 if metric else 0.0)


@pytest.mark.parametrize("recon,div", [("mc", "cleaning"), ("ppm", "cleaning"), ("mc", "fluxct"), ("ppm", "fluxct")])
@pytest.mark.parametrize("n", SIZES)
def test_rhs_and_steps_match_oracle(G, orc, n, recon, div):
    if recon == "ppm" and any(v == 2 for v in n):
        pytest.skip("PPM needs three cells on an active axis")
    for bc, metric in ((WL.PERIODIC, False), (WL.OUTFLOW, True)):
        w = _workload(n, bc, metric, sum(n) + 7 * bc)
        pb = orc.Problem(recon=int(recon == "ppm"), ct=int(div == "fluxct"), **w.problem_kwargs())
        s = G.solver_for(w, device=DEV, reconstruction=recon, divergence=div)
        P = torch.from_numpy(w.P).to(DEV)
        R, Rr = s.rhs(P).cpu().numpy(), orc.rhs(pb, w.P)
        scale = np.abs(Rr).reshape(9, -1).max(axis=1)
        err = np.abs(R - Rr).reshape(9, -1).max(axis=1) / np.maximum(scale, scale.max() * 1e-3)
        print(w.name, recon, div, bc, metric, "rhs", err.max(), flush=True)
        assert np.all(err <= 1e-11)
        U = s.cons(P)
        for _ in range(w.nsteps):
            s.step(U, w.dt)
        Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, w.nsteps)
        err = orc.parity_error(U.cpu().numpy(), Ur)
        print(w.name, recon, div, bc, metric, "steps", err.max(), flush=True)
        assert np.all(err <= 1e-10)


def test_rhs_loads_the_cache(G):
    """A right-hand side leaves the primitives (ghosts included) for the next step,
    as the conversion does."""
    w = _workload((70, 9, 5), WL.OUTFLOW, True, 3)
    P = torch.from_numpy(w.P).to(DEV)
    a, b = G.solver_for(w, device=DEV), G.solver_for(w, device=DEV)
    Ua = a.cons(P)
    Ub = Ua.clone()
    b.rhs(P)
    a.step(Ua, w.dt)
    b.step(Ub, w.dt)
    assert torch.equal(Ua, Ub)


@pytest.mark.parametrize("rk", [2, 3])
@pytest.mark.parametrize("bc", [WL.PERIODIC, WL.OUTFLOW])
@pytest.mark.parametrize("n", [2, 3, 5, 52, 53, 56, 57, 208, 209, 224, 225, 700])
def test_line_step(G, orc, n, bc, rk):
    """A whole step of a 1D grid in registers, at the edges of a wave's own cells
    (52 with RK3, 56 with RK2) and of one workgroup's (4 waves): bitwise as
    recorded, and the oracle's within its bar."""
    w = _workload((n, 1, 1), bc, False, n + rk)
    w.rk_order = rk
    P = torch.from_numpy(w.P).to(DEV)
    a, b = G.solver_for(w, device=DEV), G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
    Ua, Ub = a.cons(P), b.cons(P)
    for _ in range(3):
        a.step(Ua, w.dt)
        b.step_record(Ub, w.dt, 0)
        assert torch.equal(Ua, Ub)
    assert torch.equal(a.prim(Ua), b.prim(Ub))
    assert a.status() == b.status()
    pb = orc.Problem(**w.problem_kwargs())
    Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, 3)
    assert np.all(orc.parity_error(Ua.cpu().numpy(), Ur) <= 1e-10)


@pytest.mark.parametrize("n,bc,metric", [((64, 64, 64), WL.PERIODIC, False), ((31, 63, 127), WL.OUTFLOW, True),
                                         ((499, 8, 63), WL.OUTFLOW, False), ((30, 15, 511), WL.PERIODIC, True)])
def test_tiled_step(G, orc, n, bc, metric):
    """Grids that fill one round of the tile kernel, whole and with ragged tiles and
    segments: bitwise as recorded, and the oracle's within its bar."""
    w = _workload(n, bc, metric, sum(n))
    w.rk_order = 2
    P = torch.from_numpy(w.P).to(DEV)
    a, b = G.solver_for(w, device=DEV), G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
    Ua, Ub = a.cons(P), b.cons(P)
    for _ in range(2):
        a.step(Ua, w.dt)
        b.step_record(Ub, w.dt, 0)
        assert torch.equal(Ua, Ub)
    assert a.status() == b.status()
    pb = orc.Problem(**w.problem_kwargs())
    Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, 2)
    err = orc.parity_error(Ua.cpu().numpy(), Ur)
    print(w.name, bc, metric, err.max(), flush=True)
    assert np.all(err <= 1e-10)


@pytest.mark.parametrize("n,bc,metric", [((63, 63, 63), WL.OUTFLOW, True), ((31, 128, 63), WL.PERIODIC, True),
                                         ((96, 94, 28), WL.OUTFLOW, False), ((32, 56, 143), WL.PERIODIC, False)])
def test_ragged_tiles(G, orc, n, bc, metric):
    """Grids the tile kernel takes (the choice itself is asserted) whose last tiles
    are cut short along x or y and whose last segment has one plane: against the
    oracle, and bitwise as recorded."""
    import ctypes as C
    o = G.Opts()
    o.rk_order = 2
    assert G.load().grmhd_internal_step_kernel(C.byref(G.make_grid(n, (0,) * 3, (1,) * 3, (bc,) * 3)), C.byref(o)) == 2
    w = _workload(n, bc, metric, sum(n))
    w.rk_order = 2
    P = torch.from_numpy(w.P).to(DEV)
    a, b = G.solver_for(w, device=DEV), G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
    Ua, Ub = a.cons(P), b.cons(P)
    for _ in range(2):
        a.step(Ua, w.dt)
        b.step_record(Ub, w.dt, 0)
        assert torch.equal(Ua, Ub)
    assert a.status() == b.status()
    pb = orc.Problem(**w.problem_kwargs())
    Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, 2)
    err = orc.parity_error(Ua.cpu().numpy(), Ur)
    print(w.name, bc, metric, err.max(), flush=True)
    assert np.all(err <= 1e-10)


@pytest.mark.parametrize("n,recon,div", [((1, 1, 16384), "mc", "cleaning"), ((1, 4, 16400), "mc", "cleaning"),
                                         ((2, 3, 16390), "mc", "fluxct"), ((32, 1, 16384), "mc", "cleaning"),
                                         ((1, 1, 2048), "ppm", "cleaning"), ((3, 3, 2049), "ppm", "fluxct")])
def test_thin_planes(G, orc, n, recon, div):
    """Long grids along z of a few positions a plane take the face kernels (the choice
    itself is asserted): right-hand side, also in place, and steps against the
    oracle, bitwise as recorded."""
    import ctypes as C
    o = G.Opts()
    o.rk_order, o.reconstruction, o.divergence = 3, int(recon == "ppm"), int(div == "fluxct")
    assert G.load().grmhd_internal_step_kernel(C.byref(G.make_grid(n, (0,) * 3, (1,) * 3, (0,) * 3)), C.byref(o)) == 0
    for bc, metric in ((WL.PERIODIC, False), (WL.OUTFLOW, True)):
        w = _workload(n, bc, metric, sum(n) + 7 * bc)
        pb = orc.Problem(recon=int(recon == "ppm"), ct=int(div == "fluxct"), **w.problem_kwargs())
        s = G.solver_for(w, device=DEV, reconstruction=recon, divergence=div)
        P = torch.from_numpy(w.P).to(DEV)
        R, Rr, Q = s.rhs(P).cpu().numpy(), orc.rhs(pb, w.P), P.clone()
        scale = np.abs(Rr).reshape(9, -1).max(axis=1)
        err = np.abs(R - Rr).reshape(9, -1).max(axis=1) / np.maximum(scale, scale.max() * 1e-3)
        print(w.name, recon, div, bc, metric, "rhs", err.max(), flush=True)
        assert np.all(err <= 1e-11)
        assert np.array_equal(s.rhs(Q, Q).cpu().numpy(), R)
        U = s.cons(P)
        for _ in range(w.nsteps):
            s.step(U, w.dt)
        Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, w.nsteps)
        err = orc.parity_error(U.cpu().numpy(), Ur)
        print(w.name, recon, div, bc, metric, "steps", err.max(), flush=True)
        assert np.all(err <= 1e-10)
        if recon == "mc" and div == "cleaning":
            b = G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
            Ub = b.cons(P)
            for _ in range(w.nsteps):
                b.step_record(Ub, w.dt, 0)
            assert torch.equal(U, Ub) and torch.equal(s.prim(U), b.prim(Ub))
            # from the tape and recomputed (the primitives recovered afresh differ in last bits)
            x = torch.ones_like(U)
            b.step_adjoint_recorded(0, x)
            assert bool(torch.isfinite(x).all())
