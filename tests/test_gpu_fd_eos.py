"""Finite-difference solver: each kernel instance (base EOS x shaped or not) and meshes just below,
at and above the 40 x 24 nodes that a tile reads (remainder or compare for the periodic wrap),
against the oracle's MacCormack step, element-wise to 1e-12 as the other meshes."""
import numpy as np
import pytest

import oracle as O
from lbm_inputs import droplet_density

pytestmark = pytest.mark.gpu

PR = dict(base=1, a=2 / 49, b=2 / 21, R=1.0, omega=0.344, scale=0.25)
EOS = {
    "cs": dict(base=0, a=0.387, b=4.0, R=1.0, Tr=0.7),
    "cs-smooth": dict(base=0, a=0.387, b=4.0, R=1.0, Tr=0.7, shape=1, alpha=0.8, k_vap=2.0),
    "cs-peng": dict(base=0, a=0.387, b=4.0, R=1.0, Tr=0.7, shape=3, r_theta=0.45),
    "pr": dict(PR, Tr=0.85),
    "pr-smooth": dict(PR, Tr=0.85, shape=1, alpha=0.5, k_vap=2.0),
}


@pytest.mark.parametrize("nx,ny", [(39, 23), (40, 24), (41, 25), (64, 33)])
@pytest.mark.parametrize("kind", sorted(EOS))
def test_fd_instances_match_oracle(gpu_lib, kind, nx, ny):
    lbm = gpu_lib
    kw = EOS[kind]
    e, _ = lbm.eos_build(lbm.make_eos(**kw))
    eo, _ = O.eos_build(O.make_eos(**kw))
    rho0 = droplet_density(nx, ny, e.rho_v, e.rho_l, R=7, W=10)
    rng = np.random.default_rng(nx + ny)
    u0, v0 = 1e-3 * rng.standard_normal((ny, nx)), 1e-3 * rng.standard_normal((ny, nx))
    F = lbm.FdSolver(lbm.make_fd_params(nx, ny, e, dt=0.1, eps=e.eps, tau_e=1.1, tau_nu=0.9), rho0, u0, v0, device="cuda:0")
    F.step(40)
    F.check()
    r, u, v = (a.cpu().numpy() for a in F.fields())
    OF = O.FdSolver(O.make_fd_params(nx, ny, eo, dt=0.1, eps=eo.eps, tau_e=1.1, tau_nu=0.9))
    OF.set(rho0, u0, v0)
    OF.run(40)
    ro, uo, vo = OF.get()
    assert np.abs(r - ro).max() <= 1e-12 * np.abs(ro).max()
    assert max(np.abs(u - uo).max(), np.abs(v - vo).max()) <= 1e-12 * max(np.abs(uo).max(), np.abs(vo).max())
