"""Calls of one, two and a few steps on short periodic lattices, single and batched: each launch length
has its own kernel or its own strips, and all of them hold the same state."""
import numpy as np
import pytest

import oracle as O
from lbm_inputs import planar_density, random_field

pytestmark = pytest.mark.gpu

SMOOTH = dict(Tr=0.6, a=0.387, b=4.0, shape=1, alpha=0.834, k_vap=2 / 0.387)
CALLS = (1, 2, 1, 3, 2, 17, 1, 5)  # 32 steps


def _rho0(nx, ny, e):
    r = planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=1 if ny > nx else 0)
    return r * (1 + 0.01 * random_field(nx, ny, 1.0, 1.0, seed=nx * 1000 + ny))


@pytest.mark.parametrize("reduce_every", [0, 1, 2, 5])
@pytest.mark.parametrize("nx,ny", [(1, 1), (1024, 1), (32, 32), (89, 13), (355, 16), (15000, 4), (14999, 4), (15000, 5)])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_short_calls_hold_the_one_step_kernels_bits(gpu_lib, prec, nx, ny, reduce_every):
    """Same node arithmetic in another order: equal populations; the history's FP64 sums to rounding."""
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    rho0, out = _rho0(nx, ny, e), []
    for variant in (0, lbm.VARIANT_BLOCK):
        L = lbm.Lattice(lbm.make_params(nx, ny, e, sigma=s, prec=prec, kernel_variant=variant, reduce_every=reduce_every),
                        rho0, device="cuda:0")
        for n in CALLS:
            L.step(n)
        L.check()
        assert L.state()[0] == sum(CALLS)
        out.append((L.populations().cpu().numpy(), L.history()))
    assert np.array_equal(out[0][0], out[1][0])
    assert out[0][1].shape == out[1][1].shape and (out[0][1][:, 0] == out[1][1][:, 0]).all()
    if reduce_every:
        assert np.abs(out[0][1][:, 1:] - out[1][1][:, 1:]).max() <= 1e-12 * rho0.sum()


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["auto", "persistent", "grouped"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_short_calls_of_a_batch_match_the_oracle(gpu_lib, prec, mode):
    """Lattices cut into strips, one of them with a last strip of few columns, beside resident ones."""
    lbm = gpu_lib
    shapes = [(355, 16), (1500, 3), (7, 5), (89, 13), (1025, 1)]
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    eo, so = O.eos_build(O.make_eos(**SMOOTH))
    rhos = [_rho0(nx, ny, e) for nx, ny in shapes]
    B = lbm.Batch([lbm.make_params(nx, ny, e, sigma=s, prec=prec) for nx, ny in shapes], rhos, device="cuda:0")
    B.set_mode(mode)
    for n in CALLS:
        B.step(n)
    B.check()
    for (nx, ny), rho0, got in zip(shapes, rhos, B.macros()):
        OL = O.Lattice(O.make_params(nx, ny, eo, sigma=so))
        OL.init_eq(rho0)
        OL.run(sum(CALLS))
        m = OL.macros()
        # the bounds of the batched kernels against the oracle
        assert np.abs(got["rho"] - m["rho"]).max() <= (1e-12 if prec == lbm.FP64 else 2e-5) * m["rho"].max(), (nx, ny)
        for k in ("ux", "uy"):
            assert np.abs(got[k] - m[k]).max() <= (1e-12 if prec == lbm.FP64 else 1e-5), (nx, ny, k)
