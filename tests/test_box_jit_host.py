"""Size-specialised box kernels: the code object of a plan's kernel holds that
kernel and no other (each costs compile time in every specialisation)."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake"))


def test_code_objects_hold_one_kernel(runtime, tmp_path):
    fake_hip.run(runtime, """
import glob, os, re
cache = %r
ctypes.CDLL(None).setenv(b"TTX_JIT_CACHE", cache.encode(), 1)
plan = ttx.ttx_plan_create(ttx.F32, (2, 0, 1), (40, 36, 50))
assert ttx.ttx_plan_specialise(plan, False)
name = ttx.ttx_plan_kernel_name(plan, 0.5, 1 << 20, 3 << 20)
assert "_box" in name, name
code, = (open(f, "rb").read() for f in glob.glob(os.path.join(cache, "*.co")))
kernels = set(re.findall(rb"[A-Za-z0-9_]+(?=[.]kd)", code))
assert kernels == {name.encode()}, kernels
""" % str(tmp_path))
