"""Builds the HIP library ``libttx.so`` (gfx950) in-tree with hipcc.

Every source under ``csrc/`` is compiled to an object in ``_build/`` (in
parallel) and linked into ``paper_1607_01249_amd/libttx.so``.  Device code
is built with floating-point contraction off (Eqn. 1 is evaluated as two
rounded products and a rounded sum) and without packed-FP32 instructions.
"""
import concurrent.futures
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libttx.so")
ARCH = os.environ.get("TTX_OFFLOAD_ARCH", "gfx950")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-variable", "-ffp-contract=off",
          "-I" + CSRC, "-I" + os.path.join(os.path.dirname(HERE), "include"), "-I" + BUILD]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = ["hipcc", *COMMON]
    if src.endswith(".hip"):
        cmd += DEVICE + ["-x", "hip"]
    else:   # host-only translation units
        cmd += ["--offload-arch=" + ARCH, "-D__HIP_PLATFORM_AMD__"]
    cmd += ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    return obj


# Headers compiled at run time for size-specialised kernels (hipRTC), in
# the order they are handed to it.
JIT_HEADERS = ["device_types.h", "tile_kernels.h", "box.h", "box_kernel.h"]


def _embed_jit_headers():
    """Writes _build/ttx_jit_headers.inc: the JIT headers as string literals."""
    out = ["// generated by build.py from csrc/: the headers of the size-specialised kernels"]
    names, texts = [], []
    for i, name in enumerate(JIT_HEADERS):
        text = open(os.path.join(CSRC, name)).read()
        delim = "ttx_src"
        assert (")" + delim + '"') not in text
        # raw literals in chunks (string literal length limits), concatenated
        chunks = [text[k:k + 8000] for k in range(0, len(text), 8000)]
        texts.append("\n".join('R"%s(%s)%s"' % (delim, c, delim) for c in chunks))
        names.append('"%s"' % name)
    out.append("static const char* const kJitHeaderNames[] = {%s};" % ", ".join(names))
    out.append("static const char* const kJitHeaderSources[] = {\n%s};" % ",\n".join(texts))
    out.append("static constexpr int kJitHeaderCount = %d;" % len(JIT_HEADERS))
    path = os.path.join(BUILD, "ttx_jit_headers.inc")
    data = "\n".join(out) + "\n"
    if not os.path.exists(path) or open(path).read() != data:
        with open(path + ".tmp", "w") as f:
            f.write(data)
        os.replace(path + ".tmp", path)


def build(jobs=None, verbose=False):
    """Compiles and links the library; returns the path of libttx.so."""
    os.makedirs(BUILD, exist_ok=True)
    _embed_jit_headers()
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    jobs = jobs or min(len(srcs), os.cpu_count() or 4, 16)
    with concurrent.futures.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", "--offload-arch=" + ARCH, "-o", tmp, *objs, "-lhiprtc", "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    os.replace(tmp, LIB)
    if verbose:
        print(LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
