"""GPU adjoint (grmhd_step_adjoint, grmhd_cons_adjoint, grmhd_prim_adjoint)
against the differentiable oracle (torch.autograd over the oracle's
discretisation), element by element, and the gradient of a loss against
central finite differences of the GPU forward step.

Bar against the oracle: grouped relative L1 <= 1e-10 (FP64, the same branch
choices on both sides; the operations run in different orders)."""
import sys

import numpy as np
import pytest
import torch

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BAR = 1e-10


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def G():
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    return grmhd


@pytest.fixture(scope="module")
def AD(orc):
    from oracle import grmhd_autodiff
    return grmhd_autodiff


def _vary_all(P, amp_p=0.05, amp_phi=0.01):
    P = P.copy()
    nz, ny, nx = P.shape[1:]
    Z, Y, X = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    P[1] *= 1 + amp_p * np.sin(2 * np.pi * X / nx + 0.4) * np.cos(2 * np.pi * Y / ny + 0.2) \
        * np.cos(2 * np.pi * Z / nz + 0.7)
    P[8] = amp_phi * np.cos(2 * np.pi * Z / nz + 0.3) * np.sin(2 * np.pi * Y / ny + 0.5) \
        * np.cos(2 * np.pi * X / nx + 0.9)
    return P


def _floored_box():
    """The curved smooth box, weakly magnetised (field and Phi scaled by
    1e-6), with an atmosphere region (rho = rho_atm / 2 at rest: its interior
    cells are reset to the atmosphere) and a cold region (rho ~ 1 at rest,
    p = p_atm / 2: its interior cells' pressure is floored).  Both decisions
    are far from their thresholds, so the GPU and oracle recoveries take the
    same ones.  (Where a decision is made by rounding -- a pressure recovered
    at p_atm to within the noise of the energy cancellation, as in the
    atmosphere of the curved blob -- the two root finders may decide
    differently, and the derivative of such a cell, of size 1/p_atm, then
    differs.)"""
    w = WL.smooth_box(n=(12, 10, 8), metric=WL.ISO_SCHW, rk_order=3)
    P = w.P.copy()
    nz, ny, nx = P.shape[1:]
    Z, Y, X = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    atm = X >= 8
    cold = (X < 4) & (Y >= 6)          # apart from the atmosphere: only hot gas reaches it
    P[5:9] *= 1e-6
    P[0][atm] = 0.5 * w.rho_atm
    P[1][atm] = w.p_atm
    for v in (2, 3, 4):
        P[v][atm | cold] = 0.0
    P[1][cold] = 0.5 * w.p_atm
    w.P = P
    w.name = "floored_box"
    return w


def _cases():
    w2 = WL.config2(n=(10, 9, 8), nsteps=1)
    w2.P = _vary_all(w2.P)
    return {"periodic_flat": w2, "smooth_curved_rk3": WL.smooth_box(metric=WL.ISO_SCHW, rk_order=3),
            "floored_box": _floored_box(), "riemann_1d": WL.config1(3, n=64)}


CASES = _cases()


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def test_cons_adjoint(G, orc, AD):
    for name in ("periodic_flat", "smooth_curved_rk3"):
        w = CASES[name]
        pb = orc.Problem(**w.problem_kwargs())
        rng = np.random.default_rng(1)
        Ub = rng.standard_normal(w.P.shape)
        s = G.solver_for(w, device=DEV, adjoint=True)
        Pb = s.cons_adjoint(_t(w.P), _t(Ub)).cpu().numpy()
        P = torch.from_numpy(w.P.copy()).requires_grad_(True)
        (AD.prim2con(pb, P) * torch.from_numpy(Ub)).sum().backward()
        err = orc.parity_error(Pb, P.grad.numpy())
        say(name, "cons_adjoint rel-L1", err)
        assert np.all(err <= BAR)


def test_prim_adjoint(G, orc, AD):
    for name in ("periodic_flat", "smooth_curved_rk3", "floored_box"):
        w = CASES[name]
        pb = orc.Problem(**w.problem_kwargs())
        U0 = orc.prim2con(pb, w.P)
        rng = np.random.default_rng(2)
        Pb = rng.standard_normal(w.P.shape)
        s = G.solver_for(w, device=DEV, adjoint=True)
        Ub = s.prim_adjoint(_t(U0), _t(Pb)).cpu().numpy()
        U = torch.from_numpy(U0.copy()).requires_grad_(True)
        (AD.primitives_of(pb, U, torch.from_numpy(w.P)) * torch.from_numpy(Pb)).sum().backward()
        err = orc.parity_error(Ub, U.grad.numpy())
        say(name, "prim_adjoint rel-L1", err)
        assert np.all(err <= BAR)


@pytest.mark.parametrize("name", list(CASES))
def test_step_adjoint_matches_oracle(G, orc, AD, name):
    """One step's vector-Jacobian product, Ubar^n = (dU^(n+1)/dU^n)^T Ubar,
    by grmhd_step_adjoint (twice) and from a recorded step."""
    w = CASES[name]
    pb = orc.Problem(**w.problem_kwargs())
    U0, P0, sto = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, 1)   # a state that has been stepped
    if name == "floored_box":
        assert sto["atm"] > 0 and sto["pfloor"] > 0
    rng = np.random.default_rng(3)
    Ubar = rng.standard_normal(w.P.shape) * np.abs(U0).reshape(9, -1).mean(axis=1).reshape(9, 1, 1, 1)
    s = G.solver_for(w, device=DEV, adjoint=True)
    Ug = _t(U0)
    gpus = []
    for _ in range(2):      # the first recovery of U0 has no guess, the second a warm one
        Ub = _t(Ubar)
        s.step_adjoint(Ug, Ub, w.dt)
        gpus.append(Ub.cpu().numpy())
    st = s.status()
    # the same step recorded by a forward pass and reversed from the tape
    sr = G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
    Ur = _t(U0)
    sr.prim(Ur)
    sr.step_record(Ur, w.dt, 0)
    Ub = _t(Ubar)
    sr.step_adjoint_recorded(0, Ub)
    gpus.append(Ub.cpu().numpy())
    U = torch.from_numpy(U0.copy()).requires_grad_(True)
    P = AD.primitives_of(pb, U, torch.from_numpy(P0))
    U1, _ = AD.step(pb, U, P, w.dt, 1)
    (U1 * torch.from_numpy(Ubar)).sum().backward()
    ref = U.grad.numpy()
    bar = BAR
    if name == "floored_box":
        # the oracle against itself with the input perturbed by 1e-15 (relative)
        Un = U0 * (1 + 1e-15 * np.random.default_rng(9).standard_normal(U0.shape))
        Ux = torch.from_numpy(Un).requires_grad_(True)
        U1x, _ = AD.step(pb, Ux, AD.primitives_of(pb, Ux, torch.from_numpy(P0)), w.dt, 1)
        (U1x * torch.from_numpy(Ubar)).sum().backward()
        self_noise = float(orc.parity_error(Ux.grad.numpy(), ref).max())
        say(name, "oracle self-sensitivity", self_noise)
        bar = max(BAR, 3.0 * self_noise)
    for gpu in gpus:
        err = orc.parity_error(gpu, ref)
        say(name, "step_adjoint rel-L1", err, st)
        assert np.all(np.isfinite(gpu))
        assert np.all(err <= bar)


@pytest.mark.parametrize("name", list(CASES))
def test_recorded_step_is_the_step(G, name):
    """grmhd_step_record advances U and the primitives bitwise as grmhd_step
    does, step after step, and leaves the context ready for a plain step."""
    w = CASES[name]
    P0 = _t(w.P)
    a = G.solver_for(w, device=DEV)
    b = G.solver_for(w, device=DEV, adjoint=True, tape_steps=2)
    Ua, Ub = a.cons(P0), b.cons(P0)
    for k in range(3):
        a.step(Ua, w.dt)
        if k < 2:
            b.step_record(Ub, w.dt, k)
        else:
            b.step(Ub, w.dt)
        assert torch.equal(Ua, Ub), (name, k)
    assert torch.equal(a.prim(Ua), b.prim(Ub))


def _loss_chain(G, w, s, P0, tgt, nsteps):
    """Loss sum (rho(T) - rho_t)^2 and its gradient in the initial primitives
    by the adjoint chain cons -> steps -> prim, storing every state."""
    U = s.cons(P0)
    Us = [U.clone()]
    for _ in range(nsteps):
        s.step(U, w.dt)
        Us.append(U.clone())
    P = s.prim(U)
    r = P[0] - tgt
    L = float((r * r).sum())
    Pb = torch.zeros_like(P)
    Pb[0] = 2.0 * r
    Ub = s.prim_adjoint(U, Pb)
    for k in range(nsteps - 1, -1, -1):
        s.step_adjoint(Us[k], Ub, w.dt)
    return L, s.cons_adjoint(P0, Ub)


def test_loss_gradient_matches_oracle(G, orc, AD):
    """Gradient of the density loss after 3 RK2 steps w.r.t. all initial
    primitives: adjoint chain on the GPU against torch.autograd of the
    differentiable oracle."""
    w = CASES["periodic_flat"]
    pb = orc.Problem(**w.problem_kwargs())
    rng = np.random.default_rng(4)
    tgt = w.P[0] * (1 + 0.01 * rng.standard_normal(w.P[0].shape))
    s = G.solver_for(w, device=DEV, adjoint=True)
    L, g = _loss_chain(G, w, s, _t(w.P), _t(tgt), 3)
    P = torch.from_numpy(w.P.copy()).requires_grad_(True)
    U1, P1 = AD.step(pb, AD.prim2con(pb, P), P, w.dt, 3)
    Lr = ((P1[0] - torch.from_numpy(tgt)) ** 2).sum()
    Lr.backward()
    err = orc.parity_error(g.cpu().numpy(), P.grad.numpy())
    say("loss gradient rel-L1", err, "L", L, Lr.item())
    assert abs(L - Lr.item()) <= 1e-12 * Lr.item()
    assert np.all(err <= BAR)


def test_loss_gradient_finite_differences(G):
    """The adjoint workload at its full size (64^3 periodic, 50 RK2 steps,
    loss sum (rho(T) - rho_t)^2): directional derivatives along 32 seeded
    directions (uniform fields unperturbed) against central differences of
    the GPU forward map.  The map has kinks (MC branches, HLLE min/max) and
    the recovery's stopping rule adds steps of the size of its tolerance, so
    a difference quotient carries an error that falls with h until rounding
    of the loss takes over; the best of h = 1e-7, 1e-8, 1e-9 is taken, its
    error measured against the spread (RMS) of the 32 derivatives."""
    w = WL.config4(n=64, nsteps=50)
    s = G.solver_for(w, device=DEV, adjoint=True)
    P0 = _t(w.P)
    tgt = _t(w.extra["target"])
    L, g = _loss_chain(G, w, s, P0, tgt, w.nsteps)
    g = g.cpu().numpy()

    def loss(P):
        U = s.cons(P)
        for _ in range(w.nsteps):
            s.step(U, w.dt)
        r = s.prim(U)[0] - tgt
        return float((r * r).sum())
    ans, best = [], []
    for i in range(32):
        d = WL.direction(w, i)
        an = float((g * d).sum())
        errs = {}
        for h in (1e-7, 1e-8, 1e-9):
            fd = (loss(_t(w.P + h * d)) - loss(_t(w.P - h * d))) / (2 * h)
            errs[h] = abs(fd - an)
        ans.append(an)
        best.append(min(errs.values()))
        say("direction", i, "adjoint %.10g" % an, "abs err", {h: "%.2e" % e for h, e in errs.items()})
    scale = float(np.sqrt(np.mean(np.square(ans))))
    rel = np.array(best) / scale
    say("FD check: median %.2e, worst %.2e (relative to the RMS derivative %.4g)"
        % (np.median(rel), rel.max(), scale))
    assert np.median(rel) <= 1e-5 and rel.max() <= 1e-3


def test_autograd_evolve_with_checkpoints(G):
    """torch.autograd through evolve(): the gradient equals the plain adjoint
    chain, whatever the checkpoint interval; with the tape of recorded steps
    as well, to rounding (the recorded steps linearise
    around the primitives the forward steps used, the chain around primitives
    recovered afresh, which differ at rounding level).  Every variable is
    varied: at a uniform field the MC slopes sit on their kink, where the
    branch, and so the derivative, follows the rounding of the primitives."""
    from paper_1102_5202_amd.adjoint import evolve
    w = WL.config4(n=16, nsteps=7)
    w.P = _vary_all(w.P)
    s = G.solver_for(w, device=DEV, adjoint=True)
    st = G.solver_for(w, device=DEV, adjoint=True, tape_steps=10)
    tgt = _t(w.extra["target"])
    L, g_chain = _loss_chain(G, w, s, _t(w.P), tgt, w.nsteps)
    grads = []
    for solver in (s, st):
        for every in (1, 3, 10):
            P0 = _t(w.P).requires_grad_(True)
            P = evolve(solver, P0, w.dt, w.nsteps, every)
            loss = ((P[0] - tgt) ** 2).sum()
            loss.backward()
            assert abs(loss.item() - L) <= 1e-14 * L
            grads.append(P0.grad.clone())
    for e, g in enumerate(grads):
        rel = float((g - g_chain).abs().sum() / g_chain.abs().sum())
        say("evolve gradient vs chain", "taped" if e >= 3 else "untaped", rel)
        assert rel <= 1e-12


def test_autograd_evolve_tape_reused_in_between(G):
    """The forward pass records its last segment on the tape; when another
    evolution records over that tape before the backward pass, the backward
    pass recomputes the segment instead: both gradients still equal the plain
    adjoint chain."""
    from paper_1102_5202_amd.adjoint import evolve
    w = WL.config4(n=16, nsteps=5)
    w.P = _vary_all(w.P)
    s = G.solver_for(w, device=DEV, adjoint=True)
    st = G.solver_for(w, device=DEV, adjoint=True, tape_steps=4)
    tgt = _t(w.extra["target"])
    L, g_chain = _loss_chain(G, w, s, _t(w.P), tgt, w.nsteps)
    P0a = _t(w.P).requires_grad_(True)
    Pa = evolve(st, P0a, w.dt, w.nsteps, 4)
    P0b = (_t(w.P) * 1.001).requires_grad_(True)
    Pb = evolve(st, P0b, w.dt, w.nsteps, 4)          # records over a's last segment
    ((Pa[0] - tgt) ** 2).sum().backward()
    ((Pb[0] - tgt) ** 2).sum().backward()
    rel = float((P0a.grad - g_chain).abs().sum() / g_chain.abs().sum())
    say("tape reused in between: gradient vs chain", rel)
    assert rel <= 1e-12
    assert torch.isfinite(P0b.grad).all()


@pytest.mark.parametrize("k,axis,n", [(1, 1, 64), (3, 2, 64), (6, 2, 64), (7, 1, 64), (1, 2, 16384)])
def test_step_adjoint_of_riemann_problems_along_other_axes(G, orc, AD, k, axis, n):
    """Matter at rest beside a jump sits on the limiter's kinks, where the branch
    follows the rounding of the forward pass: a 1D problem along y or z takes the
    same order of operations as one along x (a long one along z by the face
    kernels)."""
    w = WL.config1(k, n=n, axis=axis)
    pb = orc.Problem(**w.problem_kwargs())
    U0, P0, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, 1)
    rng = np.random.default_rng(3)
    Ubar = rng.standard_normal(w.P.shape) * np.abs(U0).reshape(9, -1).mean(axis=1).reshape(9, 1, 1, 1)
    U = torch.from_numpy(U0.copy()).requires_grad_(True)
    U1, _ = AD.step(pb, U, AD.primitives_of(pb, U, torch.from_numpy(P0)), w.dt, 1)
    (U1 * torch.from_numpy(Ubar)).sum().backward()
    s = G.solver_for(w, device=DEV, adjoint=True, tape_steps=1)
    afresh, recorded, Ur = _t(Ubar), _t(Ubar), _t(U0)
    s.step_adjoint(_t(U0), afresh, w.dt)
    s.prim(Ur)
    s.step_record(Ur, w.dt, 0)
    s.step_adjoint_recorded(0, recorded)
    for got in (afresh, recorded):
        err = orc.parity_error(got.cpu().numpy(), U.grad.numpy())
        say("riemann", k, "along axis", axis, "step_adjoint rel-L1", err.max())
        assert np.all(err <= BAR)
