"""Runs host code of the library against the recording runtime of
fake_hip.cpp, in a process of its own."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBRARY = os.path.join(ROOT, "paper_1607_01249_amd", "libttx.so")

_PRELUDE = """
import ctypes, sys
sys.modules["torch"] = None       # its libraries need the real runtime
fake = ctypes.CDLL(%r, ctypes.RTLD_GLOBAL)
fake.fake_name.restype = ctypes.c_char_p
fake.fake_grid.restype = ctypes.c_uint64
fake.fake_first.restype = ctypes.c_uint32
import paper_1607_01249_amd as ttx
launches = lambda: [(fake.fake_name(i).decode(), fake.fake_grid(i), fake.fake_first(i))
                    for i in range(fake.fake_launches())]
"""


def build(directory):
    """Compiles the runtime; the path of its library."""
    out = os.path.join(str(directory), "fake_hip.so")
    cmd = ["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "paper_1607_01249_amd", "csrc"), "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", out, "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


def run(fake, code):
    """Runs `code` with `ttx`, `fake` (the runtime's own calls) and launches()."""
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests")]), FAKE_HIP_LIBRARY=LIBRARY)
    r = subprocess.run([sys.executable, "-c", _PRELUDE % fake + code], capture_output=True, text=True, timeout=300,
                       env=env, cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    return r.stdout
