"""The library's compiled device arithmetic (grmhd_device_arith: FP64 division,
square root and reciprocal square root as the kernels evaluate them, with the
device build's reciprocal and approximate-function flags) against correctly
rounded results on seeded operands spread over 80 binades: division within 2
ulp, square root within 1 ulp, reciprocal square root within 2 ulp; exact
cases stay exact."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def ulps(got, ref):
    return np.abs(got - ref) / np.spacing(np.abs(ref))


def test_division_sqrt_rsqrt_against_correct_rounding():
    from paper_1102_5202_amd import grmhd
    grmhd.load()
    rng = np.random.default_rng(11025202 + 77)
    n = 1 << 20
    x = 10.0 ** rng.uniform(-12.0, 12.0, n) * rng.uniform(1.0, 2.0, n)
    y = 10.0 ** rng.uniform(-12.0, 12.0, n) * rng.choice([-1.0, 1.0], n)
    out = grmhd.device_arith(torch.from_numpy(x).to(DEV), torch.from_numpy(y).to(DEV)).cpu().numpy()
    div, sq, rsq = out
    ref_div = x / y                                   # IEEE double division: correctly rounded
    ref_sq = np.sqrt(x)                               # correctly rounded
    ref_rsq = (1.0 / np.sqrt(x.astype(np.longdouble))).astype(np.float64)
    e_div, e_sq, e_rsq = ulps(div, ref_div), ulps(sq, ref_sq), ulps(rsq, ref_rsq)
    print("max ulp: div %.2f sqrt %.2f rsqrt %.2f; exact: div %.3f sqrt %.3f rsqrt %.3f"
          % (e_div.max(), e_sq.max(), e_rsq.max(), (e_div == 0).mean(), (e_sq == 0).mean(),
             (e_rsq == 0).mean()), flush=True)
    assert e_div.max() <= 2.0
    assert e_sq.max() <= 1.0
    assert e_rsq.max() <= 2.0


def test_exact_cases_stay_exact():
    from paper_1102_5202_amd import grmhd
    k = np.arange(1.0, 4097.0)
    x = k * k
    out = grmhd.device_arith(torch.from_numpy(x).to(DEV), torch.from_numpy(k).to(DEV)).cpu().numpy()
    assert np.array_equal(out[0], k)                  # k^2 / k
    assert np.array_equal(out[1], k)                  # sqrt of a perfect square
    p = 4.0 ** np.arange(-20, 21)
    o2 = grmhd.device_arith(torch.from_numpy(p).to(DEV), torch.from_numpy(np.ones_like(p)).to(DEV)).cpu().numpy()
    assert np.array_equal(o2[0], p)                   # x / 1
    assert np.array_equal(o2[2], 1.0 / np.sqrt(p))    # 1/sqrt of a power of 4


def test_short_forms_against_correct_rounding():
    """The FP64 path's reciprocal (either sign) and square roots over the range they
    are stated for, 1e-290 (the least argument the signal speeds' root is given) to
    1e290.  By their last operation the reciprocal and the square root are within an
    ulp (half one plus truncation of 2^-66), the reciprocal square root within two
    (its residual carries the rounding of one product)."""
    from paper_1102_5202_amd import grmhd
    L = grmhd.load()
    rng = np.random.default_rng(11025202 + 78)
    n = 1 << 20
    x = 10.0 ** rng.uniform(-290.0, 289.0, n) * rng.uniform(1.0, 10.0, n)
    x[: n // 2] = 10.0 ** rng.uniform(-12.0, 12.0, n // 2)     # where the solver's values lie
    x[:4] = [1e-290, 1e290, 1.0, 1e-16]
    sign = rng.choice([-1.0, 1.0], n)
    xt = torch.from_numpy(x * sign).to(DEV)
    out = torch.empty((3, n), dtype=torch.float64, device=DEV)
    st = torch.cuda.current_stream()
    L.grmhd_internal_roots.argtypes = [C.c_void_p, C.c_void_p, C.c_longlong, C.c_void_p]
    assert L.grmhd_internal_roots(xt.data_ptr(), out.data_ptr(), n, C.c_void_p(st.cuda_stream)) == 0
    rcp, rsq, sq = out.cpu().numpy()
    ref_rsq = (1.0 / np.sqrt(x.astype(np.longdouble))).astype(np.float64)
    e = ulps(rcp, sign / x), ulps(rsq, ref_rsq), ulps(sq, np.sqrt(x))
    print("max ulp: rcp %.2f rsqrt %.2f sqrt %.2f; exact: rcp %.3f rsqrt %.3f sqrt %.3f"
          % (*(v.max() for v in e), *((v == 0).mean() for v in e)), flush=True)
    assert e[0].max() <= 1.0
    assert e[1].max() <= 2.0
    assert e[2].max() <= 1.0
