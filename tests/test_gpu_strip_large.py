"""Strip kernel on lattices and batches whose populations take more than 64 MiB: their stores are
plain, not streaming, and hold what the one-step kernel stores."""
import numpy as np
import pytest

from lbm_inputs import planar_density, random_field

pytestmark = pytest.mark.gpu

SMOOTH = dict(Tr=0.6, a=0.387, b=4.0, shape=1, alpha=0.834, k_vap=2 / 0.387)


def _rho0(nx, ny, e):
    return planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=0) * (1 + 0.01 * random_field(nx, ny, 1.0, 1.0, seed=nx))


@pytest.mark.parametrize("prec,nx,ny", [(0, 60000, 16), (1, 60000, 16), (0, 200000, 3)])
def test_large_strip_lattices_hold_the_one_step_kernels_bits(gpu_lib, prec, nx, ny):
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    rho0, out = _rho0(nx, ny, e), []
    for variant in (0, lbm.VARIANT_BLOCK):
        P = lbm.make_params(nx, ny, e, sigma=s, prec=prec, kernel_variant=variant, reduce_every=5)
        assert 2 * lbm.layout(P)[1] > 64 << 20
        L = lbm.Lattice(P, rho0, device="cuda:0")
        L.step(11)
        L.check()
        out.append((L.populations().cpu().numpy(), L.history()))
        L.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert np.abs(out[0][1][:, 1] - out[1][1][:, 1]).max() <= 1e-12 * rho0.sum()


@pytest.mark.parametrize("width", [30000, 60000], ids=["to 256 MiB", "beyond"])
def test_large_strip_batches_match_the_one_step_kernel(gpu_lib, width):
    """1e-13 of the field's largest value, as between the batched modes.  Batches beyond 256 MiB stream
    their stores again."""
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    shapes = [(width, 16), (31, 16), (width - 1, 16)]
    rhos = [_rho0(nx, ny, e) for nx, ny in shapes]
    P = [lbm.make_params(nx, ny, e, sigma=s) for nx, ny in shapes]
    B = lbm.Batch(P, rhos, device="cuda:0")
    B.step(11)
    B.check()
    got = B.macros()
    for (nx, ny), rho0, g in zip(shapes, rhos, got):
        L = lbm.Lattice(lbm.make_params(nx, ny, e, sigma=s, kernel_variant=lbm.VARIANT_BLOCK), rho0, device="cuda:0")
        L.step(11)
        m = L.macros()
        for k in ("rho", "ux", "uy"):
            w = m[k].cpu().numpy()
            assert np.abs(g[k] - w).max() <= 1e-13 * (np.abs(w).max() + 1e-300), (nx, k)
