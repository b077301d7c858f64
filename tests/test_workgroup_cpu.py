"""Kernels of a step run on the CPU, one workgroup with its work-items one
after the other between barriers (tests/emulate): what must not depend on which
work-item comes first.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
EMU = os.path.join(HERE, "emulate")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1208_2643_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("amdclang++") or shutil.which("clang++", path="/opt/rocm/llvm/bin")
    if cxx is None:
        pytest.skip("clang++ not found")
    exe = str(tmp_path_factory.mktemp("emulate") / "workgroup")
    r = subprocess.run([cxx, "-x", "c++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-I", EMU,
                        "-I", CSRC, os.path.join(EMU, "workgroup.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]

    def call(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout.split()
    return call


@pytest.mark.parametrize("wave", range(8))
def test_rising_stop_flag_leaves_no_tile_half_done(driver, wave):
    """The stop flag may rise in the launch whose tiles look at it, here once the
    first wave of a workgroup has looked: the workgroup runs whole or not at all,
    and leaves the copy of u that it read."""
    wrote, read = driver("tile", wave)
    assert wrote in ("all", "none") and read == "kept"


@pytest.mark.parametrize("m,n", [(2, 2), (4, 4), (8, 8), (16, 16), (32, 32), (4, 2), (8, 16),
                                 (32, 16)])
@pytest.mark.parametrize("bc", [0, 3])
def test_persistent_levels_do_not_depend_on_the_order_of_the_lanes(driver, m, n, bc):
    """A cycle over the levels of one workgroup, work-items first to last and last
    to first: the same bits.  (Levels of up to 128 cells run in one wave, whose lanes
    are ordered by fences only.)"""
    diff, size = map(float, driver("coarse", m, n, bc))
    assert diff == 0.0 and size > 0.0


@pytest.mark.parametrize("pivot", [0, 1])
@pytest.mark.parametrize("h,c,al,amp,seed", [
    (45.2, 3.03e6, 0.0, 2.25e-6, 20), (13.8, 5.32e8, 0.0, 5.40e-5, 773),
    (21.5, 7.39e6, 0.0, 1.99e-5, 146), (0.8, 0.02, 0.4, 1.0, 1)])
def test_coarsest_newton_stops_within_its_tolerance(driver, pivot, h, c, al, amp, seed):
    """Large dt (c), alpha = 0 and a small phi: a step's square says little about the
    error it leaves.  Against the same solve with every step taken: the tolerance,
    1e-15 of 1 + |phi|, beside what rounding moves that solve by from step to step
    (1e-14 where the elimination with pivoting is ill conditioned)."""
    err, noise, size = map(float, driver("newton", h, c, al, amp, pivot, seed))
    assert err <= 1e-15 * (1.0 + size) + noise


@pytest.mark.parametrize("norms,most", [(1, 1), (3, 100), (224, 300), (225, 100000), (101, 100)])
def test_readback_takes_the_recorded_norms_only(driver, norms, most):
    """Of a history with room for every allowed cycle the host gets the norms that the
    step recorded, behind the 32 doubles of state and sums."""
    written, wrong = map(int, driver("readback", norms, most))
    assert written == 32 + norms and wrong == 0
