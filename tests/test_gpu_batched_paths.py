"""Batches on each of their paths: lattices cut into strips beside resident ones, against the oracle, and
graphs of grouped two-step launches, captured and replayed."""
import numpy as np
import pytest

import oracle as O
from lbm_inputs import droplet_density, droplet_on_film, planar_density, random_field

pytestmark = pytest.mark.gpu

SMOOTH = dict(Tr=0.6, a=0.387, b=4.0, shape=1, alpha=0.834, k_vap=2 / 0.387)
TAU = [1.0, 1.1, 1.2, 1.0, 1.1, 1.0, 1.1, 0.8, 0.8]

# a tall resident lattice, strips of several heights (the last one of 1135 x 4 has one column in launches
# of 8 steps), a small resident lattice
CUT = [(12, 60), (1135, 4), (355, 16), (513, 2), (9, 9)]


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_cut_and_resident_lattices_match_the_oracle(gpu_lib, prec):
    """Full launches and shorter ones; the bounds of the batched kernels against the oracle."""
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    eo, so = O.eos_build(O.make_eos(**SMOOTH))
    rhos = [planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=1 if ny > nx else 0)
            * (1 + 0.01 * random_field(nx, ny, 1.0, 1.0, seed=nx)) for nx, ny in CUT]
    B = lbm.Batch([lbm.make_params(nx, ny, e, sigma=s, tau=TAU, prec=prec) for nx, ny in CUT], rhos, device="cuda:0")
    for n in (8, 80, 21, 5):
        B.step(n)
    B.check()
    for (nx, ny), rho0, got in zip(CUT, rhos, B.macros()):
        OL = O.Lattice(O.make_params(nx, ny, eo, sigma=so, tau=TAU))
        OL.init_eq(rho0)
        OL.run(114)
        m = OL.macros()
        assert np.abs(got["rho"] - m["rho"]).max() <= (1e-12 if prec == lbm.FP64 else 2e-5) * m["rho"].max(), (nx, ny)
        for k in ("ux", "uy"):
            assert np.abs(got[k] - m[k]).max() <= (1e-12 if prec == lbm.FP64 else 1e-5), (nx, ny, k)


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_grouped_graphs_replay_the_captured_launches(gpu_lib, prec, walls):
    """A lattice that the strip kernel refuses keeps the batch on grouped two-step launches: 128 steps
    captured, then replayed, from either buffer, and a tail; equal bits however the calls are split."""
    lbm = gpu_lib
    e, s = lbm.eos_build(lbm.make_eos(**SMOOTH))
    if walls:
        kw = dict(walls=True, rho_wall_lo=e.rho_l, rho_wall_hi=e.rho_v)
        rhos = [droplet_on_film(64, 40, e.rho_v, e.rho_l, R=8, h=6, gap=3, V=0.0, W=6)[0]]
        P = [lbm.make_params(64, 40, e, sigma=s, tau=TAU, prec=prec, **kw)]
    else:
        rhos = [droplet_density(130, 37, e.rho_v, e.rho_l, R=10, W=6)]
        P = [lbm.make_params(130, 37, e, sigma=s, tau=TAU, prec=prec)]
    for nx, ny in ((300, 4), (62, 4)):
        P.append(lbm.make_params(nx, ny, e, sigma=s, tau=TAU, prec=prec))
        rhos.append(planar_density(nx, ny, e.rho_v, e.rho_l, W=10, axis=0))
    out = []
    # 128-step graphs from both buffers and replays of each (an odd number of launches flips the buffer)
    for calls in ((128, 128, 2, 256, 128, 7), (649,)):
        B = lbm.Batch(P, rhos, device="cuda:0")
        B.set_mode(lbm.BATCH_GROUPED)
        for n in calls:
            B.step(n)
        B.check()
        out.append(B.macros())
    persistent = lbm.Batch(P, rhos, device="cuda:0")
    persistent.set_mode(lbm.BATCH_PERSISTENT)
    persistent.step(649)
    persistent.check()
    for a, b, c in zip(out[0], out[1], persistent.macros()):
        for k in ("rho", "ux", "uy"):
            assert np.array_equal(a[k], b[k]), k
            if prec == lbm.FP64:  # the node arithmetic of the other mode: as test_batched_modes_agree
                assert np.abs(a[k] - c[k]).max() <= 1e-13 * (np.abs(c[k]).max() + 1e-300), k
