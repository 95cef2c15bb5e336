"""Short and small periodic lattices: many steps per launch, populations in LDS (lbm_strip.h).

Against the oracle in FP64, against the one-step row block in FP32: lattices resident in one
workgroup (1 node to 1024, one column, one row), strips with one and many workgroups, a last
strip of one column, 1 to 16 rows, launches that end at a reduction, several calls in a row.
"""
import numpy as np
import pytest

import oracle as O
from lbm_inputs import planar_density, random_field

pytestmark = pytest.mark.gpu

TAU_MRT = [1.0, 1.1, 1.25, 1.0, 1.15, 1.0, 1.15, 0.8, 0.8]
SMOOTH = dict(Tr=0.6, a=0.387, b=4.0, shape=1, alpha=0.834, k_vap=2 / 0.387)
#         resident                                            | strips
SHAPES = [(1, 1), (1, 7), (2, 200), (200, 2), (32, 32), (1024, 1), (1025, 1), (2, 513), (513, 2), (1500, 3), (355, 16),
          (89, 13)]


def _rho0(nx, ny, e):
    r = planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=1 if ny > nx else 0)
    return r * (1 + 0.01 * random_field(nx, ny, 1.0, 1.0, seed=nx * 1000 + ny))


def _params(lbm, nx, ny, prec, **kw):
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    vt = dict(var_tau=True, tau_l=0.8, tau_v=1.4) if nx % 2 else {}
    return e, s, vt, lbm.make_params(nx, ny, e, sigma=s, tau=TAU_MRT, prec=prec, reduce_every=7, **vt, **kw)


@pytest.mark.parametrize("nx,ny", SHAPES)
def test_strip_fp64_matches_oracle(gpu_lib, nx, ny):
    """Element-wise 1e-12 of the largest population, as every FP64 kernel: the node arithmetic is
    the same, in another order."""
    lbm = gpu_lib
    e, s, vt, P = _params(lbm, nx, ny, lbm.FP64)
    rho0 = _rho0(nx, ny, e)
    L = lbm.Lattice(P, rho0, device="cuda:0")
    eo, so = O.eos_build(O.make_eos(**SMOOTH))
    OL = O.Lattice(O.make_params(nx, ny, eo, sigma=so, tau=TAU_MRT, **vt))
    OL.init_eq(rho0)
    mass = rho0.sum()
    for n in (1, 2, 30, 8):
        L.step(n)
        OL.run(n)
        L.check()
        g, o = L.populations().cpu().numpy(), OL.get_f()
        assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max(), n
    h = L.history()
    assert h[:, 0].tolist() == [0, 7, 14, 21, 28, 35]
    assert np.abs(h[:, 1] - mass).max() <= 1e-12 * mass
    assert np.abs(h[:, 2:]).max() <= 1e-12 * mass  # a periodic lattice at rest keeps zero momentum


@pytest.mark.parametrize("nx,ny", SHAPES)
def test_strip_fp32_matches_row_block(gpu_lib, nx, ny):
    """Against the one-step kernel: 1e-6 of the largest deviation per step, and each node's mass
    exact in both (FP64 sums of the same values)."""
    lbm = gpu_lib
    e, _, _, P = _params(lbm, nx, ny, lbm.FP32_SHIFTED)
    _, _, _, Q = _params(lbm, nx, ny, lbm.FP32_SHIFTED, kernel_variant=lbm.VARIANT_BLOCK)
    rho0 = _rho0(nx, ny, e)
    A, B = lbm.Lattice(P, rho0, device="cuda:0"), lbm.Lattice(Q, rho0, device="cuda:0")
    done = 0
    for n in (1, 19, 9):
        A.step(n)
        B.step(n)
        done += n
        A.check()
        a, b = A.populations().cpu().numpy(), B.populations().cpu().numpy()
        dev = np.abs(b - b.min()).max()
        assert np.abs(a - b).max() <= 1e-6 * done * dev, n
    ha, hb = A.history(), B.history()
    assert (ha[:, 0] == hb[:, 0]).all()
    assert np.abs(ha[:, 1] - hb[:, 1]).max() <= 1e-9 * np.abs(hb[:, 1]).max()


def test_strip_launch_split_does_not_matter(gpu_lib):
    """The state between launches is the one LDS holds: any split of the steps gives the same bits."""
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    for nx, ny in ((200, 2), (1500, 3)):
        out = []
        for split in ((60,), (1, 3, 16, 33, 7)):
            L = lbm.Lattice(lbm.make_params(nx, ny, e, sigma=s), planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=0))
            for n in split:
                L.step(n)
            out.append(L.populations().cpu().numpy())
        assert np.array_equal(*out)


def test_strip_reports_the_first_unstable_step(gpu_lib):
    """The step of the first bad density, in the middle of a launch and beside a strip's edge, is
    the one the one-step kernels name."""
    lbm = gpu_lib
    ep, _ = lbm.eos_build(lbm.make_eos(base=1, a=2 / 49, b=2 / 21, omega=0.344, Tr=0.5))
    for nx, ny in ((64, 4), (1500, 3)):
        rho0 = planar_density(nx, ny, ep.rho_v, ep.rho_l, W=2, axis=0)
        said = []
        for variant in (0, lbm.VARIANT_BLOCK):
            L = lbm.Lattice(lbm.make_params(nx, ny, ep, kernel_variant=variant), rho0, device="cuda:0")
            L.step(400)
            with pytest.raises(lbm.LbmError) as ei:
                L.check()
            said.append(str(ei.value))
        assert said[0] == said[1]
