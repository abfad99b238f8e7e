"""2D FP64 grids whose planes are too large for the sweep's 32-bit offsets take the
face kernels and the update in place: a plane of 2^28 cells made of 256 copies of a
64-row strip steps as the strip does (which is swept), with MC and with PPM.  Bar:
that of either against the oracle, relative L1 1e-10 a row, and 1e-9 of a row's
largest value everywhere, so that no misplaced cell passes."""
import numpy as np
import pytest
import torch

from paper_1102_5202_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NX, STRIP, COPIES = 1 << 14, 64, 256


@pytest.mark.parametrize("recon", ["mc", "ppm"])
def test_large_plane_steps_as_its_strip(recon):
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    # workspace (cache, stage state, two face arrays), primitives and U
    if torch.cuda.mem_get_info()[0] < 6.5 * 72 * NX * STRIP * COPIES:
        pytest.skip("needs 126 GB of GPU memory")
    rng = np.random.default_rng(5)
    base = torch.tensor([1.0, 0.2, 0.2, -0.15, 0.1, 0.15, 0.1, -0.1, 0.02], dtype=torch.float64, device=DEV)
    noise = torch.from_numpy(rng.uniform(-0.3, 0.3, (9, 1, STRIP, NX))).to(DEV)
    P = base.view(9, 1, 1, 1) * (1.0 + noise)
    dx = 1.0 / NX

    def solver(ny):
        return grmhd.Solver((NX, ny, 1), (0.0,) * 3, (1.0, ny * dx, 1.0), (WL.PERIODIC,) * 3, gamma=4.0 / 3.0,
                            rk_order=2, reconstruction=recon, device=DEV)

    small = solver(STRIP)
    Us = small.cons(P)
    Rs = small.rhs(P)
    large = solver(STRIP * COPIES)
    X = P.repeat(1, 1, COPIES, 1)

    def same(big, ref, what):
        for v in range(9):
            r = ref[v, 0]
            d = (big[v, 0].view(COPIES, STRIP, NX) - r).abs_()
            scale = float(r.abs().max())
            assert float(d.max()) <= 1e-9 * scale, (what, v)
            assert float(d.sum()) <= 1e-10 * COPIES * float(r.abs().sum()) + 1e-14 * scale, (what, v)

    large.rhs(X, X)
    same(X, Rs, "rhs")
    for v in range(9):
        X[v, 0].view(COPIES, STRIP, NX).copy_(P[v, 0])
    U = large.cons(X)
    del X
    for _ in range(2):
        small.step(Us, 0.2 * dx)
        large.step(U, 0.2 * dx)
    same(U, Us, "step")
    assert large.status()["fail"] == 0
