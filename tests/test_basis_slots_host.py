"""The byte budget of the stored BiCGStab basis, with and without slots taken ahead (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("slots") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_0910_1048_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "basis_slots_driver.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("fp64", [0, 4, 40, 1000])
@pytest.mark.parametrize("budget", [10, 22, 100, 150, 200, 1000])
@pytest.mark.parametrize("pool", [0, 1, 30, 2000])
def test_slots_taken_ahead_do_not_move_the_budget(driver, fp64, budget, pool):
    """With a pool of an earlier FP64 solve, slots for the FP32 phase are taken ahead while the iterations are still
    in FP64: they hold FP32 vectors and count as such."""
    def solve(ahead):
        r = subprocess.run([driver, str(fp64), str(budget), str(pool), str(ahead)], capture_output=True, text=True,
                           check=True)
        return r.stdout.split()
    plain, ahead = solve(0), solve(64)
    assert ahead[:2] == plain[:2]
    assert int(ahead[2]) <= int(plain[2])   # and no buffer more is allocated
