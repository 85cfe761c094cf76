"""The operand loads of the contraction kernels on the CPU: for random
contractions (one to three labels a group, any storage orders, extents that
are whole tiles and units and odd ones), both types and every tile shape, each
lane's reads of each tile and step, formed by the kernel's own code, lie inside
the operand."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def contract_sim(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("contract")
    csrc = os.path.join(ROOT, "paper_1607_01249_amd", "csrc")
    exe, obj = str(tmp / "contract_sim"), str(tmp / "contract_sim.o")
    flags = ["-O2", "-std=c++17", "-I" + csrc, "-I" + os.path.join(ROOT, "include")]
    for cmd in (["hipcc", *flags, "-x", "hip", "--cuda-host-only", "-c", os.path.join(ROOT, "tests", "contract_sim.cpp"),
                 "-o", obj],
                ["hipcc", *flags, "-D__HIP_PLATFORM_AMD__", obj, os.path.join(csrc, "contract_plan.cpp"), "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("seed", [1, 2])
def test_loads_stay_inside_the_operands(contract_sim, seed):
    r = subprocess.run([contract_sim, str(seed), "60"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    m = re.match(r"ok: 60 contractions, (\d+) whole-unit plans, (\d+) with 80 columns along their run, "
                 r"(\d+) lanes in the walk and (\d+) beyond\n", r.stdout)
    assert m and all(int(x) > 0 for x in m.groups()), r.stdout
