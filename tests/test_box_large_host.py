"""Box tiles of four units a thread on the CPU (problems of 10^5 elements and
more, all eight types, both beta classes, leading dimensions): bounds, values
and coverage, as in test_box_host.py."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def box_sim_large(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("box") / "box_sim_large")
    csrc = os.path.join(ROOT, "paper_1607_01249_amd", "csrc")
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + csrc, "-I" + os.path.join(ROOT, "include"),
           "-I/opt/rocm/include", "-x", "c++", os.path.join(ROOT, "tests", "box_sim_large.cpp"),
           os.path.join(csrc, "box_plan.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("seed", [1, 2])
def test_four_units_a_thread(box_sim_large, seed):
    r = subprocess.run([box_sim_large, str(seed), "80"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    m = re.fullmatch(r"ok: four units a thread, by type( 10){8}, (\d+) with remainders\n", r.stdout)
    assert m and int(m.group(2)) > 0, r.stdout
