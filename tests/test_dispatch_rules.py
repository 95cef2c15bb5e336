"""The dispatch rules of the library's headers (host code), compiled into a small program and called on
sizes: which launches the strip kernel takes, how much of its work is recomputed columns, and which
two-step tiles are timed."""
import os
import shutil
import subprocess

import pytest

from paper_2107_06355_amd import build as B

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <vector>
#include "lbm.h"
#include "lbm_device.h"
#include "lbm_strip.h"
using namespace lbmk;
// one line in: precision, steps, lattices, then nx ny of each; steps 0: the two-step tiles of the first
// lattice, rows and waves of the library's pick and then of every timed candidate
int main()
{
    int prec, steps, n;
    while (std::scanf("%d %d %d", &prec, &steps, &n) == 3) {
        std::vector<lbm_params> p(n);
        for (auto& q : p) {
            q = lbm_params();
            q.prec = prec;
            if (std::scanf("%d %d", &q.nx, &q.ny) != 2) return 1;
        }
        if (steps == 0) {
            const TwoStepShape pick = run_shape(p[0]);
            std::printf("%d %d", pick.rows, pick.waves);
            p[0].tile_rows = -1;
            TwoStepShape c[kMaxShapes];
            const int k = two_step_candidates(p[0], c);
            for (int i = 0; i < k; ++i) std::printf(" %d %d", c[i].rows, c[i].waves);
            std::printf("\n");
            continue;
        }
        const StripPlan s = strip_plan(n, p.data());
        std::printf("%d %d %d", s.threads, s.steps, (int)strip_runs(p[0], steps));
        for (auto& q : p)
            std::printf(" %d %d", s.threads ? strip_cols(q, s.threads) : 0, s.threads ? strip_out(q, s.threads, steps) : 0);
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(lines) -> the program's output, a list of numbers per line."""
    if shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.hip", d / "rules"
    src.write_text(PROGRAM)
    subprocess.check_call([B.HIPCC, *B.FLAGS, "-w", "-x", "hip", "-I" + os.path.join(B.ROOT, "include"), "-I" + B.CSRC,
                           str(src), "-o", str(exe)])

    def run(lines):
        text = "".join("%s\n" % " ".join(str(v) for v in ln) for ln in lines)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        got = [[int(v) for v in ln.split()] for ln in out.splitlines()]
        assert len(got) == len(lines)
        return got

    return run


@pytest.mark.parametrize("prec", [0, 1])
def test_short_launches_of_a_lattice_leave_the_strip_kernel(rules, prec):
    """One and two steps run on the one- and two-step kernels, but for wide lattices of up to 4 rows."""
    shapes = [(1, 1), (200, 2), (1024, 1), (32, 32), (1500, 3), (4096, 16), (65536, 16), (14999, 4), (15000, 5),
              (15000, 4), (500000, 1)]
    lines = [(prec, n, 1, nx, ny) for nx, ny in shapes for n in (1, 2, 3, 16)]
    for (_, n, _, nx, ny), got in zip(lines, rules(lines)):
        assert got[0] > 0, (nx, ny)  # every one of them has a plan
        assert got[2] == (n > 2 or (ny <= 4 and nx >= 15000)), (nx, ny, n)


@pytest.mark.parametrize("prec", [0, 1])
def test_strips_recompute_only_the_columns_a_launch_uses_up(rules, prec):
    """A strip of n steps advances all but 2 n - 1 columns on each side, whatever the plan's most steps."""
    for nx, ny in [(1500, 3), (355, 16), (4096, 16), (65536, 16), (2048, 4)]:
        threads, steps = rules([(prec, 1, 1, nx, ny)])[0][:2]
        assert steps >= 3
        for n in range(1, steps + 1):
            cols, out = rules([(prec, n, 1, nx, ny)])[0][3:]
            assert cols == threads // ny and out == cols - 2 * (2 * n - 1), (nx, ny, n)


@pytest.mark.parametrize("prec", [0, 1])
def test_timed_tiles_include_the_one_that_runs_untimed(rules, prec):
    """tile_rows = -1 times, among others, the height that tile_rows = 0 runs; each shape once."""
    sizes = [(1400, 225), (384, 785), (100, 2580)] if prec == 0 else [(249, 2196), (211, 2695)]
    sizes += [(nx, ny) for nx in range(60, 2500, 83) for ny in range(60, 2500, 97)]
    picks = set()
    for (nx, ny), got in zip(sizes, rules([(prec, 0, 1, nx, ny) for nx, ny in sizes])):
        pick, cand = tuple(got[:2]), list(zip(got[2::2], got[3::2]))
        assert pick in cand and len(set(cand)) == len(cand) <= 8, (nx, ny, got)
        if len(cand) > 1:
            picks.add(pick[0])
            assert set(range(7, 11) if prec == 0 else [10] + list(range(14, 19))) <= {r for r, _ in cand}, (nx, ny, got)
    assert picks & ({5, 6} if prec == 0 else {12})  # heights outside the timed range were among them


@pytest.mark.parametrize("prec", [0, 1])
def test_the_batches_tested_against_the_oracle_are_cut(rules, prec):
    """What tests/test_gpu_batched_paths.py relies on: strips of 8 steps, with a last one of one column,
    beside resident lattices."""
    from test_gpu_batched_paths import CUT

    sizes = [v for s in CUT for v in s]
    assert rules([(prec, 8, len(CUT), *sizes)])[0][1] == 8
    got = rules([(prec, 8, len(CUT), *sizes)])[0][3:]
    cols, out = got[0::2], got[1::2]
    cut = [c < nx for (nx, _), c in zip(CUT, cols)]
    assert cut == [False, True, True, True, False]
    assert CUT[1][0] % out[1] == 1
