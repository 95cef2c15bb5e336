"""The device EOS at the ends of its branches: the end of an ellipse (a square root of zero) and a pole
of the base EOS (a division by zero)."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _loop_eos(lbm):
    """A Smooth loop whose ellipses end at 0.375 and 0.875: 1 - (rho - knot)^2 / a^2 is zero there."""
    e, _ = lbm.eos_build(lbm.make_eos(Tr=0.7))
    e.shape = lbm.SHAPE_SMOOTH
    e.rho_v, e.rho_max, e.rho_min, e.rho_l = 0.25, 0.5, 0.75, 0.96
    e.p_max, e.p_min, e.b1, e.b3 = 0.01, 0.001, 0.005, 0.002
    e.a1sq = e.a3sq = 0.125 ** 2
    return e


# the ends, and densities inside each ellipse and the cubic between them
LOOP = [0.375, 0.4375, 0.5, 0.625, 0.75, 0.8125, 0.875]


# FP64: an FP64 lattice's density is a rounded sum of its populations, so not the ends
@pytest.mark.parametrize("prec,rho", [(1, r) for r in LOOP] + [(0, r) for r in LOOP[1:-1]])
def test_the_end_of_an_ellipse_is_an_ordinary_density(gpu_lib, prec, rho):
    """A uniform lattice stays as it is: p of the EOS, no instability."""
    lbm = gpu_lib
    e = _loop_eos(lbm)
    P = lbm.make_params(70, 40, e, prec=prec, rho_ref=rho)
    L = lbm.Lattice(P, np.full((40, 70), rho), device="cuda:0")
    L.step(4)
    L.check()
    m = L.macros()
    want = lbm.load().lbm_eos_pressure(C.byref(e), rho)
    assert np.isfinite(want)
    assert np.abs(m["p"].cpu().numpy() - want).max() <= 4e-15 * max(e.p_max, abs(want))


@pytest.mark.parametrize("rho", LOOP)
def test_the_end_of_an_ellipse_in_the_finite_difference_solver(gpu_lib, rho):
    lbm = gpu_lib
    F = lbm.FdSolver(lbm.make_fd_params(40, 30, _loop_eos(lbm)), np.full((30, 40), rho))
    F.step(3)
    F.check()
    r, u, v = (a.cpu().numpy() for a in F.fields())
    assert (r == rho).all() and (u == 0).all() and (v == 0).all()


@pytest.mark.parametrize("base", ["cs", "pr"])
def test_a_pole_of_the_base_eos_has_infinite_pressure(gpu_lib, base):
    """C-S at 4/b, P-R at 1/b: p is infinite, psi zero, and the lattice unstable, as with IEEE division."""
    lbm = gpu_lib
    kw = dict(base=lbm.BASE_CS, b=4.0, a=0.5) if base == "cs" else dict(base=lbm.BASE_PR, b=0.125, a=2 / 49, omega=0.344)
    e, _ = lbm.eos_build(lbm.make_eos(Tr=0.7, **kw))
    rho = 1.0 if base == "cs" else 8.0
    L = lbm.Lattice(lbm.make_params(64, 8, e, prec=lbm.FP32_SHIFTED, rho_ref=rho), np.full((8, 64), rho), device="cuda:0")
    import torch

    p, psi = (torch.zeros((8, 64), dtype=torch.float64, device="cuda:0") for _ in range(2))
    rc = lbm.load().lbm_macros(L._h, None, None, None, psi.data_ptr(), p.data_ptr(), None, None, None, L._s())
    assert rc == lbm.LBM_EUNSTABLE
    assert np.isposinf(p.cpu().numpy()).all() and (psi.cpu().numpy() == 0).all()
