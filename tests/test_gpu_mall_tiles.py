"""Two-step tiles with two rows per wave on both sides of the sizes where the kernel changes (both
buffers within 64 MiB, within 256 MiB, beyond): the same populations as the one-step kernel, bit for
bit (the node arithmetic is the same, whichever rows load)."""
import numpy as np
import pytest

from lbm_inputs import droplet_density

pytestmark = pytest.mark.gpu

EOS = dict(base=0, a=0.387, b=4.0, Tr=0.6, shape=1, alpha=0.834, k_vap=2 / 0.387)
STEPS = 5
# nodes x 80 B (FP32) or 144 B (FP64): just under and just over 64 and 256 MiB; last bands of one row and of all
SIZES = {"fp32": [(1201, 685), (1201, 703), (1855, 1801), (1855, 1819)],
         "fp64": [(1201, 379), (1201, 391), (1405, 1321), (1405, 1330)]}


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec_name,nx,ny", [(p, *s) for p in SIZES for s in SIZES[p]])
def test_two_rows_per_wave_equal_one_step(gpu_lib, prec_name, nx, ny, walls):
    lbm = gpu_lib
    prec = lbm.FP64 if prec_name == "fp64" else lbm.FP32_SHIFTED
    e, s = lbm.eos_build(lbm.make_eos(**EOS))
    rho0 = droplet_density(nx, ny, e.rho_v, e.rho_l, R=0.45 * ny, W=8)
    kw = dict(walls=True, rho_wall_lo=e.rho_v, rho_wall_hi=e.rho_v) if walls else {}
    out = []
    for more in (dict(tile_rows=18 if prec == lbm.FP32_SHIFTED else 10), dict(kernel_variant=lbm.VARIANT_BLOCK)):
        L = lbm.Lattice(lbm.make_params(nx, ny, e, sigma=s, tau=[1.0] * 7 + [0.7] * 2, prec=prec, **more, **kw), rho0,
                        device="cuda:0")
        L.step(STEPS)
        L.check()
        out.append(L.populations().cpu().numpy())
        L.close()
    assert np.array_equal(*out)
