"""The tile height of the two-step transposed kernel: where the pick changes (10, 12 or 14 waves per
workgroup while every tile has a compute unit, else 16), periodic and walled, its gradients are those
of the 16-wave tiles, which a workspace without room for the smaller tiles' accumulators still runs.
The node arithmetic does not depend on the height, so dL/drho0 is the same up to how a compiler
contracts it (4 ulp of its largest value per step); the sums differ in the order of their partial
sums (n ulp of the sum of the terms' magnitudes, which the largest gradient bounds up to the factor
their signs cancel by: 1e4 here)."""
import numpy as np
import pytest

from lbm_inputs import droplet_density

pytestmark = pytest.mark.gpu

EOS = dict(base=0, a=0.387, b=4.0, Tr=0.6, shape=1, alpha=0.834, k_vap=2 / 0.387)
STEPS = 4
CUS = 256
# one strip of 58 columns or two, one band or two; 6 strips: 42 bands of 4, 6 and 8 rows
SIZES = [(58, 25), (59, 24), (117, 41), (300, 168), (300, 169), (300, 252), (300, 253), (300, 336)]


def _tiles(nx, ny, waves):
    return -(-nx // 58) * -(-ny // (waves - 6))


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec_name", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_smaller_tiles_give_the_same_gradients(gpu_lib, nx, ny, prec_name, walls):
    lbm = gpu_lib
    prec = lbm.FP64 if prec_name == "fp64" else lbm.FP32_SHIFTED
    e, s = lbm.eos_build(lbm.make_eos(**EOS))
    rho0 = droplet_density(nx, ny, e.rho_v, e.rho_l, R=0.3 * min(nx, ny), W=4)
    kw = dict(walls=True, rho_wall_lo=e.rho_v, rho_wall_hi=e.rho_v) if walls else {}
    waves = next((w for w in (10, 12, 14) if _tiles(nx, ny, w) <= CUS), 16)
    # accumulators: 10 per workgroup of the larger grid, the one-step kernel's (62 columns, 10 rows) or this one's
    one = -(-nx // 62) * -(-ny // 10)
    kb = [-(-80 * max(one, _tiles(nx, ny, w)) // 256) for w in (waves, 16)]
    assert waves < 16 and kb[0] > kb[1]  # a byte less than the layout asks for still holds the 16-wave tiles'
    out = []
    for less in (0, 1):
        L = lbm.Lattice(lbm.make_params(nx, ny, e, sigma=s, prec=prec, **kw), rho0, device="cuda:0")
        L.enable_recording(STEPS)
        L.step(STEPS)
        L._adj = L._adj[: L._adj.numel() - less]
        g = L.adjoint(rho0 - rho0.mean(), want_rho0=True)
        out.append((g.pop("rho0").cpu().numpy(), np.array([g[n] for n in lbm.GRAD_NAMES])))
        L.close()
    (r, v), (r16, v16) = out
    ulp = np.finfo(np.float64 if prec == lbm.FP64 else np.float32).eps
    assert np.isfinite(r).all() and np.abs(r).max() > 0
    assert np.abs(r - r16).max() <= 4 * STEPS * ulp * np.abs(r16).max()
    assert np.abs(v - v16).max() <= 1e4 * 4 * STEPS * ulp * np.abs(v16).max()
