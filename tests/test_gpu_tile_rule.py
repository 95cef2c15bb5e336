"""The two-step tile height the library picks for a lattice (tile_rows = 0): where the pick changes,
on both sides, periodic and walled, it runs the same populations as the tallest tile, bit for bit
(the node arithmetic does not depend on the height), and the same reductions up to the order of
their partial sums."""
import numpy as np
import pytest

from lbm_inputs import droplet_density

pytestmark = pytest.mark.gpu

EOS = dict(base=0, a=0.387, b=4.0, Tr=0.6, shape=1, alpha=0.834, k_vap=2 / 0.387)
# 58-column strips x bands: one workgroup per CU or more (256 tiles), one round or more (512), few
# tiles or many (about a thousand), two rows per wave for many tiles (2000 and 2600 of 18 rows)
SIZES = [(100, 70), (464, 320), (465, 321), (522, 341), (696, 426), (754, 440), (930, 690), (1160, 1799), (1161, 1801),
         (1450, 1872), (1451, 1873)]


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec_name", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_picked_height_runs_the_same_steps(gpu_lib, nx, ny, prec_name, walls):
    lbm = gpu_lib
    prec = lbm.FP64 if prec_name == "fp64" else lbm.FP32_SHIFTED
    e, s = lbm.eos_build(lbm.make_eos(**EOS))
    rho0 = droplet_density(nx, ny, e.rho_v, e.rho_l, R=0.2 * min(nx, ny), W=8)
    kw = dict(walls=True, rho_wall_lo=e.rho_v, rho_wall_hi=e.rho_v) if walls else {}
    out = []
    for h in (0, 18 if prec == lbm.FP32_SHIFTED else 10):
        P = lbm.make_params(nx, ny, e, sigma=s, tau=[1.0] * 7 + [0.7] * 2, prec=prec, reduce_every=5, tile_rows=h, **kw)
        L = lbm.Lattice(P, rho0, device="cuda:0")
        L.step(13)
        L.check()
        out.append((L.populations().cpu().numpy(), L.history(), L.tile_shape()))
        L.close()
    (f, hist, shape), (g, hist_g, _) = out
    rows, waves = shape
    assert (rows, waves) in [(10, 16)] + [(r, 12) for r in range(11, 19)] if prec == lbm.FP32_SHIFTED else (5 <= rows <= 10 and waves == 8)
    assert np.array_equal(f, g)
    assert np.array_equal(hist[:, 0], hist_g[:, 0])
    assert np.abs(hist - hist_g)[:, 1:].max() <= 1e-13 * hist_g[:, 1].max()
