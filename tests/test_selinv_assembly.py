"""Assembly of sparse-direct fronts below which pads leave nothing to add: on
one-tier stacks a box whose surroundings are all pads has an empty update set.
On the host the reads of the assembly are checked against the fronts' blocks
(tests/cpp/selinv_assembly_check.cpp); on the GPU such stacks are compared with
the oracle's selected inversion.  Both sides are float64 direct methods on
stacks below 3e3 nodes, so the bar is 1e-11 as for the other small stacks."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import selinv as osel
from paper_2607_05818_amd import gen

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_05818_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_assembly_reads_stay_inside_the_fronts(tmp_path):
    exe = str(tmp_path / "selinv_assembly_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-o", exe,
                    os.path.join(HERE, "cpp", "selinv_assembly_check.cpp"),
                    os.path.join(CSRC, "selinv_plan.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all ok" in r.stdout


def _tier(seed, nx, ny, pads):
    rng = np.random.default_rng(seed)
    return gen.make_desc(1, nx, ny, rng.uniform(0.5, 2, ny * (nx - 1)), rng.uniform(0.5, 2, (ny - 1) * nx),
                         np.zeros((0, 2), dtype=np.int32), np.zeros((0, 0)), pads)


# one pad on a chain; pads on the root's wall (x = nx / 2), on it and on a wall
# of each half, and on every second column
EMPTY_SETS = [(67, 1, [[50, 0]]), (40, 1, [[20, 0], [10, 0], [31, 0]]),
              (31, 16, [[15, y] for y in range(16)]),
              (70, 33, [[35, y] for y in range(33)] + [[x, 16] for x in range(70)]),
              (33, 9, [[x, y] for x in range(0, 33, 2) for y in range(9)])]


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,pads", EMPTY_SETS)
def test_empty_update_sets(nx, ny, pads):
    from paper_2607_05818_amd import reff
    d = _tier(nx, nx, ny, pads)
    print("[case] selinv empty update sets", nx, ny, flush=True)
    want = osel.diag_full(d)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_selinv_diag(h)
    h.close()
    free = want > 0
    assert np.all(got[~free] == 0.0)
    assert np.max(np.abs(got[free] - want[free]) / want[free]) <= 1e-11


@pytest.mark.gpu
def test_empty_update_sets_in_a_forest():
    from paper_2607_05818_amd import reff
    plans = [_tier(nx, nx, ny, pads) for nx, ny, pads in EMPTY_SETS]
    plans.insert(2, gen.small_random_desc(5, 3, 20, 17, 30, 3))
    print("[case] selinv empty update sets, forest", flush=True)
    outs, _ = reff.reff_selinv_batch(plans)
    for d, got in zip(plans, outs):
        want = osel.diag_full(d)
        free = want > 0
        assert np.all(got[~free] == 0.0)
        assert np.max(np.abs(got[free] - want[free]) / want[free]) <= 1e-11
