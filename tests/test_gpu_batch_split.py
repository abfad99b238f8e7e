"""The split placement of the batched ensemble at the edges of its walk: a wave
updates 60 cells at a time and a workgroup 240, in problems packed whole and
in problems divided into parts, against the CPU oracle run alone."""
import numpy as np
import pytest

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
EDGES = [3, 4, 59, 60, 61, 62, 120, 121, 239, 240, 241, 242, 300, 301, 480, 481, 482]


def _ensemble(lengths, bc, k):
    """Shock tubes of the given lengths, four steps each (a different count for every third)."""
    parts = [WL.config5(nprob=1, nmin=n, nmax=n, k=k + i) for i, n in enumerate(lengths)]
    e = WL.Ensemble(name="edges", P=[p.P[0] for p in parts], n=[p.n[0] for p in parts],
                    dt=[p.dt[0] for p in parts], steps=[4 + (i % 3 == 0) for i in range(len(parts))])
    e.bc = bc
    return e


# FP64 rounding over five steps of a shock tube: the bar of the ensemble's own tests
BAR = 1e-10


@pytest.mark.parametrize("bc", [WL.PERIODIC, WL.OUTFLOW])
@pytest.mark.parametrize("lengths", [EDGES * 16, EDGES, [1201, 1440, 1441]], ids=["packed", "mixed", "parted"])
def test_split_edges_match_oracle(orc, lengths, bc):
    from paper_1102_5202_amd import grmhd
    e = _ensemble(lengths, bc, 11)
    s = grmhd.batch_for(e, device=DEV)
    s.set_shape(256, 2)
    U = s.cons(s.pack(e.P))
    s.evolve(U)
    Us = s.unpack(U.cpu())
    for b in range(min(len(lengths), len(EDGES))):
        w = e.problem(b)
        pb = orc.Problem(**w.problem_kwargs())
        Ur, _, _ = orc.step(pb, orc.prim2con(pb, w.P), w.P, w.dt, w.nsteps)
        err = orc.parity_error(Us[b].numpy(), Ur.reshape(9, -1))
        print("split", bc, "n", e.n[b], err.max(), flush=True)
        assert np.all(err <= BAR), (b, e.n[b], err)
