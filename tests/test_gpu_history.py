"""The reduction history's ring (4096 rows) as the host reads it: before, at and past its end, all
rows or the newest few, in order; and lbm_macros' sums beside the error word."""
import numpy as np
import pytest

from lbm_inputs import planar_density

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [5, 4096, 4100, 8195])
def test_history_ring(gpu_lib, steps):
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(Tr=0.7))
    rho0 = planar_density(64, 2, e.rho_v, e.rho_l, W=8, axis=0)
    L = lbm.Lattice(lbm.make_params(64, 2, e, sigma=s, reduce_every=1), rho0, device="cuda:0")
    L.step(steps)
    for rows in (10000, 4096, 7, 0):
        h = L.history(rows)
        n = min(steps, 4096, rows)
        assert h[:, 0].tolist() == list(range(steps - n, steps))
        assert np.abs(h[:, 1] - rho0.sum()).max(initial=0.0) <= 1e-12 * rho0.sum()
    assert abs(L.mass_momentum()[0] - rho0.sum()) <= 1e-12 * rho0.sum()
