"""lbm_layout's workspace holds its parts and nothing beside them (host logic only)."""
import os
import re

import pytest

from paper_2107_06355_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("nx,ny,prec", [(1, 1, 0), (130, 37, 1), (512, 512, 0), (2048, 1024, 1)])
def test_the_workspace_is_the_sum_of_its_parts(nx, ny, prec):
    """The error word with lbm_macros' sums, an FP64 triple per wave of the row march, a triple per block
    of the two-pass reduction, the history ring."""
    src = open(os.path.join(ROOT, "paper_2107_06355_amd", "csrc", "lbm_step.hip")).read()
    blocks, ring = (int(re.search(r"constexpr int %s = (\d+);" % k, src).group(1)) for k in ("kRedBlocks", "kHistCap"))
    e, s = lbm.eos_build(lbm.make_eos(Tr=0.7))
    P = lbm.make_params(nx, ny, e, sigma=s, prec=prec, kernel_variant=lbm.VARIANT_MARCH)
    _, _, waves = lbm.describe(P)
    assert lbm.layout(P)[2] == 256 + -(-waves * 24 // 256) * 256 + blocks * 24 + ring * 32
