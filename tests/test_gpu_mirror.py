"""Mirror images of a supersonic flow with a strong density contrast.  Where every
signal at a face runs one way the flux is exactly the upwind state's, so the
update of a mirrored state is the mirrored update to the last bit, whichever way
the flow goes: in particular the thin gas beside a dense one takes no rounding
of the dense side's flux.  For every FP64 kernel that solves faces in the
regrouped form: the sweep's right-hand side and step, the tiled step, the
ensemble."""
import numpy as np
import pytest
import torch

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# rows of U that change sign under a mirror of axis 0, 1, 2 (momentum and field along it)
FLIP = {0: (2, 5), 1: (3, 6), 2: (4, 7)}


@pytest.fixture(scope="module")
def G():
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    return grmhd


def _supersonic(n, seed):
    """Cold gas streaming towards lower indices along every active axis, its
    density (and pressure) jumping by up to seven decades between cells."""
    rng = np.random.default_rng(seed)
    shape = (n[2], n[1], n[0])
    P = np.zeros((9,) + shape)
    P[0] = 10.0 ** -rng.integers(0, 8, shape)
    P[1] = 1e-3 * P[0]
    for a in range(3):
        if n[a] > 1:
            P[2 + a] = -3.0 * (1.0 + 0.01 * rng.uniform(-1.0, 1.0, shape))
            P[5 + a] = 1e-6 * rng.uniform(-1.0, 1.0, shape)
    P[8] = 1e-9 * rng.uniform(-1.0, 1.0, shape)
    return WL.Workload(name="stream_%dx%dx%d" % n, P=P, n=n, lo=(0.0,) * 3, hi=(1.0,) * 3, bc=(WL.PERIODIC,) * 3,
                       gamma=5.0 / 3.0, rk_order=2, dt=0.2 * WL.cfl_dt(n, (0.0,) * 3, (1.0,) * 3), nsteps=1,
                       metric=WL.FLAT, M=0.0, rho_atm=1e-14, p_atm=1e-20)


def _mirror(A, axis):
    B = torch.flip(A, dims=(A.dim() - 1 - axis,)).contiguous()
    for v in FLIP[axis]:
        B[v] = -B[v]
    return B


@pytest.mark.parametrize("n", [(70, 1, 1), (40, 21, 1), (1, 30, 9), (21, 18, 10), (64, 64, 64)])
def test_mirrored_flow_is_bitwise_mirrored(G, n):
    w = _supersonic(n, sum(n))
    s = G.solver_for(w, device=DEV)
    P = torch.from_numpy(w.P).to(DEV)
    R = s.rhs(P).clone()
    U = s.cons(P)
    s.step(U, w.dt)
    assert bool(torch.isfinite(U).all())
    for axis in range(3):
        if n[axis] == 1:
            continue
        Pm = _mirror(P, axis)
        Rm = s.rhs(Pm)
        # equal as numbers (0 = -0)
        assert bool((Rm == _mirror(R, axis)).all()), (n, axis, "rhs", float((Rm - _mirror(R, axis)).abs().max()))
        Um = s.cons(Pm)
        s.step(Um, w.dt)
        assert bool((Um == _mirror(U, axis)).all()), (n, axis, "step", float((Um - _mirror(U, axis)).abs().max()))


def test_mirrored_ensemble_is_bitwise_mirrored():
    from paper_1102_5202_amd import grmhd
    ws = [_supersonic((n, 1, 1), n) for n in (59, 130, 241, 700)]
    e = WL.Ensemble(name="stream", P=[w.P.reshape(9, -1) for w in ws], n=[w.n[0] for w in ws],
                    dt=[w.dt for w in ws], steps=[2] * len(ws))
    e.bc = WL.PERIODIC
    m = WL.Ensemble(name="mirrored", P=[_mirror(torch.from_numpy(w.P), 0).numpy().reshape(9, -1) for w in ws], n=e.n,
                    dt=e.dt, steps=e.steps)
    m.bc = WL.PERIODIC
    out = []
    for x in (e, m):
        s = grmhd.batch_for(x, device=DEV)
        s.set_shape(256, 2)
        U = s.cons(s.pack(x.P))
        s.evolve(U)
        out.append(s.unpack(U.cpu()))
    for a, b in zip(*out):
        a = _mirror(a.reshape(9, 1, 1, -1), 0).reshape(9, -1)
        assert bool(torch.isfinite(a).all()) and bool((a == b.reshape(9, -1)).all()), float((a - b).abs().max())
