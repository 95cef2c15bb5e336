"""What the library says it runs, and the names bench.py gives the kernels it times: on both sides of
every bound, and kernels that the library holds (host logic only)."""
import os
import re
import shutil
import subprocess

import pytest

import bench
from paper_2107_06355_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F32, F64 = lbm.FP32_SHIFTED, lbm.FP64

CASES = [
    # nx, ny, precision, walls, tile shape -> kernel, steps per launch
    # two rows per wavefront: 64 and 256 MiB of populations are the bounds
    ((2048, 409, F32, True, (16, 12)), ("k_step2_rows2<float, 0, true, true>", 2)),
    ((2048, 410, F32, True, (16, 12)), ("k_step2_rows2_mall<float, true>", 2)),
    ((2048, 1024, F32, True, (16, 12)), ("k_step2_rows2_mall<float, true>", 2)),
    ((2048, 1638, F32, False, (18, 12)), ("k_step2_rows2_mall<float, false>", 2)),
    ((2048, 1639, F32, False, (18, 12)), ("k_step2_rows2<float, 0, false, false>", 2)),
    ((1024, 455, F64, False, (10, 8)), ("k_step2_rows2<double, 0, false, true>", 2)),
    ((1024, 456, F64, False, (10, 8)), ("k_step2_rows2_mall<double, false>", 2)),
    ((1024, 1820, F64, True, (10, 8)), ("k_step2_rows2_mall<double, true>", 2)),
    ((1024, 1821, F64, True, (10, 8)), ("k_step2_rows2<double, 0, true, false>", 2)),
    # one row per wavefront has no instance of its own for that range
    ((2048, 1024, F32, True, (10, 16)), ("k_step2_blk<float, 0, true, false>", 2)),
    ((512, 512, F32, False, (10, 16)), ("k_step2_blk<float, 0, false, true>", 2)),
]


@pytest.fixture(scope="module")
def eos():
    return lbm.eos_build(lbm.make_eos(Tr=0.7))


def _params(eos, nx, ny, prec, walls=False, **kw):
    e, s = eos
    if walls:
        kw.update(walls=True, rho_wall_lo=e.rho_l, rho_wall_hi=e.rho_v)
    return lbm.make_params(nx, ny, e, sigma=s, prec=prec, **kw)


def _strips(eos):
    out = []
    for nx, ny, prec in [(200, 2, F64), (32, 32, F32), (1024, 1, F64), (1500, 3, F32), (4096, 16, F32), (65536, 16, F64)]:
        P = _params(eos, nx, ny, prec)
        threads, steps = lbm.describe_strip(P)
        assert threads and steps >= 2
        out.append((P, threads, steps))
    return out


@pytest.mark.parametrize("case,want", CASES)
def test_two_step_instances_by_size(eos, case, want):
    nx, ny, prec, walls, shape = case
    assert bench.launched_kernel(lbm, _params(eos, nx, ny, prec, walls), shape) == want


def test_bounds_are_the_librarys():
    src = open(os.path.join(ROOT, "paper_2107_06355_amd", "csrc", "lbm_device.h")).read()
    for name, value in (("kStreamBytes", bench.STREAM_BYTES), ("kMallBytes", bench.MALL_BYTES)):
        m = re.search(r"constexpr size_t %s = \(size_t\)(\d+) << (\d+);" % name, src)
        assert value == int(m.group(1)) << int(m.group(2))


def test_strip_lattices_are_named(eos):
    for P, threads, steps in _strips(eos):
        name, n = bench.launched_kernel(lbm, P)
        nt = 2 * lbm.layout(P)[1] <= bench.STREAM_BYTES
        m = re.fullmatch(r"k_strip<(float|double), (\d+), false, (true|false)>", name)
        assert m and n == steps and (m.group(3) == "true") == nt and (m.group(1) == "float") == (P.prec == F32)
        cap = int(m.group(2))
        assert threads <= cap and (cap == 256 or 2 * threads > cap)


def test_no_strips_but_for_short_periodic_lattices_left_to_the_library(eos):
    for P in (_params(eos, 1500, 17, F64), _params(eos, 33, 32, F64), _params(eos, 1500, 3, F32, walls=True),
              _params(eos, 1500, 3, F32, kernel_variant=lbm.VARIANT_BLOCK2), _params(eos, 1500, 3, F32, tile_rows=-1),
              _params(eos, 1500, 3, F64, tile_rows=10)):
        assert lbm.describe_strip(P) == (0, 0)
    assert lbm.describe_strip(_params(eos, 1500, 16, F64))[0] > 0
    P = _params(eos, 4, 4, F64)
    P.nx = 0
    with pytest.raises(lbm.LbmError):
        lbm.describe_strip(P)


def test_the_named_kernels_are_in_the_library(eos):
    if shutil.which("nm") is None:
        pytest.skip("nm not available")
    out = subprocess.run(["nm", "-C", lbm.LIB_PATH], capture_output=True, text=True, check=True).stdout
    held = set(re.findall(r"__device_stub__(\S+<[^>]*>)\(", out))
    names = {want[0] for _, want in CASES} | {bench.launched_kernel(lbm, P)[0] for P, _, _ in _strips(eos)}
    assert names <= held, sorted(names - held)
