"""A right-hand side written over its own primitives (R = P, or the two arrays
overlapping in part) is the one written elsewhere, through a context and through
the entry point without allocation, in every combination of options and active
axes.  Both routes evaluate the same faces; the bar between them is the one of
either against the oracle, 1e-11 of a row's largest value (mixed precision:
FP32 fluxes loaded the same way, equal bits)."""
import numpy as np
import pytest
import torch

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def G():
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    return grmhd


def _workload(n, bc, metric, seed):
    rng = np.random.default_rng(seed)
    base = np.array([1.0, 0.2, 0.2, -0.15, 0.1, 0.15, 0.1, -0.1, 0.02])
    P = base[:, None, None, None] * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, (9, n[2], n[1], n[0])))
    lo, hi = ((2.0, 1.0, 1.5), (4.0, 3.0, 3.5)) if metric else ((0.0,) * 3, (1.0,) * 3)
    return WL.Workload(name="rough_%dx%dx%d" % n, P=P, n=n, lo=lo, hi=hi, bc=(bc,) * 3, gamma=4.0 / 3.0, rk_order=3,
                       dt=0.5 * WL.cfl_dt(n, lo, hi), nsteps=1, metric=WL.ISO_SCHW if metric else WL.FLAT,
                       M=1.0 if metric else 0.0)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("recon,div", [("mc", "cleaning"), ("ppm", "cleaning"), ("mc", "fluxct"), ("ppm", "fluxct")])
@pytest.mark.parametrize("n", [(300, 1, 1), (1, 70, 1), (90, 33, 1), (1, 20, 30), (40, 22, 18)])
def test_rhs_in_place(G, n, recon, div, precision):
    for bc, metric in ((WL.PERIODIC, False), (WL.OUTFLOW, True)):
        w = _workload(n, bc, metric, sum(n))
        opts = dict(precision=precision, reconstruction=recon, divergence=div)
        P = torch.from_numpy(w.P).to(DEV)
        ref = G.solver_for(w, device=DEV, **opts).rhs(P)
        bar = ref.abs().amax(dim=(1, 2, 3), keepdim=True) * (0.0 if precision == "mixed" else 1e-11)
        bar = torch.maximum(bar, bar.max() * 1e-3)
        total = P.numel()
        for shift in (0, 1, n[0] * n[1] * n[2] + 3, -5):
            for noalloc in (False, True):
                buf = torch.zeros(2 * total, dtype=torch.float64, device=DEV)
                at = max(0, -shift)
                Q = buf[at:at + total].view(P.shape)
                R = buf[at + shift:at + shift + total].view(P.shape)
                Q.copy_(P)
                if noalloc:
                    G.rhs_noalloc_for(w, Q, R=R, **opts)
                else:
                    s = G.solver_for(w, device=DEV, **opts)
                    s.rhs(Q, R)
                assert bool(((R - ref).abs() <= bar).all()), (n, bc, shift, noalloc, float((R - ref).abs().max()))
        # the primitives are in the cache for the next step
        a, b = G.solver_for(w, device=DEV, **opts), G.solver_for(w, device=DEV, **opts)
        Ua = a.cons(P)
        Ub, Q = Ua.clone(), P.clone()
        b.rhs(Q, Q)
        a.step(Ua, w.dt)
        b.step(Ub, w.dt)
        assert torch.equal(Ua, Ub)
