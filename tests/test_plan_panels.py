"""The plan data that the LDS-panel kernels read (inverse row maps, panel prefixes, wave
tasks, update matrices kept in LDS, workgroup steps, scratch sizes) against the front tree,
for both element sizes, by a host program (plan_check.cpp) over sizes, couplings and tunings."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    csrc = os.path.join(HERE, "..", "paper_1908_08292_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", os.path.join(HERE, "plan_check.cpp"),
                           os.path.join(csrc, "plan.cpp"), "-o", exe])
    return exe


def run(exe, *args):
    p = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=120)
    return p.stdout.strip()


@pytest.mark.parametrize("d,bc,sizes", [(2, 0, (2, 3, 4, 7, 8, 10, 13, 16, 17, 20, 24, 27, 32, 33, 34, 36, 38, 40, 41, 43)),
                                        (2, 1, (3, 8, 16, 24, 31, 33, 40, 47, 48, 56, 64)),
                                        (3, 0, (2, 3, 4)), (3, 1, (2, 3, 4))])
def test_default_plans(plan_check, d, bc, sizes):
    for n in sizes:
        assert run(plan_check, d, n, bc, 0, 64) == "panels", n


@pytest.mark.parametrize("leaf", [1, 4, 8, 9, 12, 32, 64, 4096])
@pytest.mark.parametrize("wave", [0, 32, 64])
def test_tuned_plans(plan_check, leaf, wave):
    for d, n, bc in ((2, 8, 0), (2, 16, 0), (2, 21, 0), (2, 32, 1), (2, 37, 0), (2, 43, 0), (3, 4, 0)):
        got = run(plan_check, d, n, bc, leaf, wave)
        assert got in ("panels", "global"), (d, n, bc, got)


def test_first_sizes_with_global_fronts(plan_check):
    for d, n in ((2, 44), (2, 47), (3, 5)):
        assert run(plan_check, d, n, 0, 0, 64) == "global"
