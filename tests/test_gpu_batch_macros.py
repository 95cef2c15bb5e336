"""Batch.macros brings its fields to the host in one copy or in three: what lbm_macros_batched wrote."""
import ctypes as C

import numpy as np
import pytest

from lbm_inputs import planar_density

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(7, 3)], [(120, 16), (45, 2)], [(1365, 64)], [(1366, 64)], [(1000, 300), (3, 5)]],
                         ids=["tiny", "small", "2 MiB", "over 2 MiB", "large"])
def test_batch_macros_on_both_sides_of_the_one_copy_bound(gpu_lib, shapes):
    lbm = gpu_lib
    import torch

    e, s = lbm.eos_build(lbm.make_eos(Tr=0.7))
    B = lbm.Batch([lbm.make_params(nx, ny, e, sigma=s) for nx, ny in shapes],
                  [planar_density(nx, ny, e.rho_v, e.rho_l, W=8, axis=0) for nx, ny in shapes], device="cuda:0")
    B.step(9)
    n = sum(nx * ny for nx, ny in shapes)
    dev = [torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    assert lbm.load().lbm_macros_batched(B._h, *[d.data_ptr() for d in dev], C.c_void_p(B.stream.cuda_stream)) == 0
    want = [d.cpu().numpy() for d in dev]
    first = B.macros()
    kept = [{k: v.copy() for k, v in m.items()} for m in first]
    B.step(3)
    B.macros()  # a later call leaves earlier results alone
    off = 0
    for (nx, ny), m, c in zip(shapes, first, kept):
        for k, w in zip(("rho", "ux", "uy"), want):
            assert np.array_equal(m[k], w[off:off + nx * ny].reshape(ny, nx)), (nx, ny, k)
            assert np.array_equal(m[k], c[k]), (nx, ny, k)
        off += nx * ny
