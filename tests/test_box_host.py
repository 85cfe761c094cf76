"""Box tiles on the CPU: the planner's boxes for random problems (orders,
leading dimensions, all eight types, odd extents), every unit of every thread
carried out with the kernel's own offsets.  Checked are the bounds of A, B and
LDS, that each element of B comes from the element of A that the definition
names, and that no two boxes write one element."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def box_sim(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("box") / "box_sim")
    csrc = os.path.join(ROOT, "paper_1607_01249_amd", "csrc")
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + csrc, "-I" + os.path.join(ROOT, "include"),
           "-I/opt/rocm/include", "-x", "c++", os.path.join(ROOT, "tests", "box_sim.cpp"),
           os.path.join(csrc, "box_plan.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("seed", [1, 2])
def test_boxes_of_random_problems(box_sim, seed):
    r = subprocess.run([box_sim, str(seed), "600"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    m = re.fullmatch(r"ok: (\d+) boxes of 600 problems, (\d+) filled, (\d+) skewed, (\d+) small\n", r.stdout)
    assert m, r.stdout
    assert all(int(x) > 0 for x in m.groups()), r.stdout
