"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values.  Lists are written as text ("160,160,64,32").
Four kinds, each through the public entry points of the Python binding:

  call         one transposition of Eqn. 1 by ``ttx.transpose``: no plan, no tuning
  plan         one by a plan that the program keeps, with its size-specialised kernel
  batch        many uneven transpositions in one persistent launch
  contraction  a binary tensor contraction with a workspace that the program keeps

Tensors are flat column-major storage; values are uniform in [-1, 1), the
distribution of the workloads that the tests and the benchmark use.
"""
import math

import numpy as np
import torch

import paper_1607_01249_amd as ttx
import workloads

_TORCH = {"f32": torch.float32, "f64": torch.float64, "c32": torch.complex64, "c64": torch.complex128}
_CODE = {"f32": ttx.F32, "f64": ttx.F64, "c32": ttx.C32, "c64": ttx.C64}
_BYTES = {"f32": 4, "f64": 8, "c32": 8, "c64": 16}
# (A's type, B's type) of every type name: one type for both, or the mixed-precision pairs
_PAIRS = {"f32": ("f32", "f32"), "f64": ("f64", "f64"), "c32": ("c32", "c32"), "c64": ("c64", "c64"),
          "sd": ("f32", "f64"), "ds": ("f64", "f32"), "cz": ("c32", "c64"), "zc": ("c64", "c32")}
_DEVICE = "cuda:0"


def _transposition(name, kind, types, size, perm, alpha, beta, outer_a="", outer_b="", alpha_im=0.0, beta_im=0.0):
    case = dict(kind=kind, types=types, size=size, perm=perm, alpha=alpha, beta=beta, alpha_im=alpha_im,
                beta_im=beta_im, outer_a=outer_a, outer_b=outer_b)
    return dict(case, name=name) if name else case


def _contraction(name, dtype, labels_a, labels_b, labels_c, extents, alpha, beta):
    case = dict(kind="contraction", types=dtype, labels_a=labels_a, labels_b=labels_b, labels_c=labels_c,
                extents=extents, alpha=alpha, beta=beta)
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest call: a few microseconds, launch and host time only.
        _transposition("call_tiny_f32", "call", "f32", "24,20,9", "2,0,1", 1.3, 0.7),
        # A small 3D tensor (3.9 MB) turned round, as between two steps of a tensor program.
        _transposition("call_3d_f32", "call", "f32", "96,128,80", "2,1,0", 1.0, 0.0),
        # Odd extents in every index, the stride-1 index only 7 long (62 MB).
        _transposition("call_odd_extents_f32", "call", "f32", "7,1023,33,65", "1,2,3,0", -0.5, 1.0),
        # A sub-tensor of a larger tensor on both sides: packing with leading dimensions.
        _transposition("call_subtensor_f64", "call", "f64", "384,96,48,32", "1,0,2,3", -0.5, 1.0,
                       "400,100,48,32", "100,400,50,32"),
        # The large 4D reversal (200 MiB), B overwritten.
        _transposition("call_4d_f32", "call", "f32", "160,160,64,32", "3,2,1,0", 1.3, 0.0),
        # A large 6D transposition that keeps its short stride-1 index, as an update.
        _transposition("call_6d_f64_kept_rows", "call", "f64", "20,16,16,20,16,16", "0,5,1,4,2,3", 1.3, 0.7),
        # Complex elements with complex scalars, 5D (200 MiB).
        _transposition("call_5d_c32", "call", "c32", "44,32,24,32,24", "1,3,0,4,2", 0.75, -0.5,
                       alpha_im=-1.25, beta_im=0.375),
        # A shape that a program repeats, with its kernel compiled for the sizes: 6D reversal, odd extents.
        _transposition("plan_6d_f32", "plan", "f32", "24,21,20,18,17,17", "5,4,3,2,1,0", 1.3, 0.7),
        # 512 uneven transpositions in one launch (4.2 GB in all).
        dict(name="batch_512", kind="batch", count=512, draw=4, max_elements=4194304),
        # A contraction whose matrix product dominates: m = n = k = 1600.
        _contraction("contract_gemm_f32", "f32", "2,4,0,5", "5,3,4,1", "0,1,2,3", "40,40,40,40,40,40", 1.0, 0.0),
        # A short sum and a large result (729 MiB), accumulated.
        _contraction("contract_short_sum_f32", "f32", "2,6,0,4", "5,3,6,1", "0,1,2,3,4,5",
                     "24,24,24,24,24,24,16", 1.0, 0.5),
        # The same in double precision, small: 96 x 64 x 512 from a sum of 8.
        _contraction("contract_short_sum_f64", "f64", "1,3,0", "3,2", "0,1,2", "96,64,512,8", -1.5, 1.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _extents(rng, total, n):
    """n extents whose product is about `total`, split by a flat Dirichlet draw (extents of one can come up)."""
    w = [rng.gammavariate(1.0, 1.0) for _ in range(n)]
    return [max(1, int(round(total ** (x / sum(w))))) for x in w]


def _text(values):
    return ",".join(str(int(v)) for v in values)


def _draw_transposition(rng):
    types = rng.choice(["f32"] * 6 + ["f64"] * 4 + ["c32", "c64", "sd", "ds", "cz", "zc"])
    ta, tb = _PAIRS[types]
    while True:
        n = rng.randint(2, 6)
        size = _extents(rng, _log(rng, 4096, 210e6 / max(_BYTES[ta], _BYTES[tb])), n)
        if np.prod([float(s) for s in size]) * max(_BYTES[ta], _BYTES[tb]) <= 220e6:
            break
    perm = rng.sample(range(n), n)
    outer_a = outer_b = ""
    if rng.random() < 0.25:
        outer_a = _text(s + rng.randint(0, 9) for s in size)
        outer_b = _text(size[k] + rng.randint(0, 9) for k in perm)
        if np.prod([float(x) for x in outer_a.split(",")]) + np.prod([float(x) for x in outer_b.split(",")]) > 1.2e8:
            outer_a = outer_b = ""   # many short indices: the padding would outweigh the tensor
    cx = tb in ("c32", "c64")
    beta = rng.choice([0.0, 0.7])
    return _transposition("", "plan" if rng.random() < 0.2 else "call", types, _text(size), _text(perm), 1.3, beta,
                          outer_a, outer_b, -1.25 if cx else 0.0, 0.375 if cx and beta else 0.0)


def _draw_contraction(rng):
    dtype = "f32" if rng.random() < 0.7 else "f64"
    while True:
        m, n, k = _log(rng, 32, 14000), _log(rng, 32, 14000), _log(rng, 4, 2048)
        size_m, size_n, size_k = (_extents(rng, x, rng.randint(1, most)) for x, most in ((m, 3), (n, 3), (k, 2)))
        m, n, k = (float(np.prod(s)) for s in (size_m, size_n, size_k))
        w = _BYTES[dtype]
        if m * n * w <= 400e6 and m * k * w <= 200e6 and n * k * w <= 200e6 and m * n * k * w <= 16.4e9:
            break
    ext = size_m + size_n + size_k
    a, b, c = len(size_m), len(size_n), len(size_k)
    lm, ln, lk = range(a), range(a, a + b), range(a + b, a + b + c)
    shuffled = [rng.sample(x, len(x)) for x in ([*lm, *lk], [*ln, *lk], [*lm, *ln])]
    return _contraction("", dtype, *(_text(x) for x in shuffled), _text(ext), 1.25, rng.choice([0.0, 0.5]))


def draw(rng):
    x = rng.random()
    if x < 0.55:
        return _draw_transposition(rng)
    if x < 0.65:
        return dict(kind="batch", count=int(_log(rng, 16, 500)), draw=rng.randrange(1 << 20),
                    max_elements=int(_log(rng, 65536, 4194304)))
    return _draw_contraction(rng)


def _ints(text):
    return [int(x) for x in text.split(",")] if text else None


def _elements(size):
    return int(np.prod([int(s) for s in size], dtype=np.int64))


def _uniform(n, dtype, gen):
    if dtype in ("c32", "c64"):
        return torch.view_as_complex(_uniform(2 * n, "f32" if dtype == "c32" else "f64", gen).view(-1, 2))
    return torch.rand(n, dtype=_TORCH[dtype], device=_DEVICE, generator=gen).mul_(2).sub_(1)


def _scalars(case):
    """alpha and beta as a program passes them: floats, or complex numbers for the complex types."""
    if _PAIRS[case["types"]][1] in ("c32", "c64"):
        return complex(case["alpha"], case["alpha_im"]), complex(case["beta"], case["beta_im"])
    return case["alpha"], case["beta"]


class _Kept:
    """A library handle that the program keeps, destroyed with it."""

    def __init__(self, handle, destroy):
        self.handle, self._destroy = handle, destroy

    def __del__(self):
        self._destroy(self.handle)


def _transposition_inputs(case, gen):
    ta, tb = _PAIRS[case["types"]]
    size, perm = _ints(case["size"]), _ints(case["perm"])
    A = _uniform(_elements(_ints(case["outer_a"]) or size), ta, gen)
    B = _uniform(_elements(_ints(case["outer_b"]) or size), tb, gen)
    return A, B, size, perm


def _batch_problems(case):
    """The batched workload's problems; |beta| <= 1, so that updates repeated on the same tensors stay finite."""
    probs = workloads.batched_problems(case["count"], case["draw"], max_elems=case["max_elements"])
    return [dict(p, beta=p["beta"] / 2, types="f32" if p["dtype"] == np.float32 else "f64") for p in probs]


def _batch_inputs(case, gen):
    """The problems, and per type the inputs and outputs: slices of one tensor each, on 256-byte boundaries."""
    probs, total = _batch_problems(case), {"f32": 0, "f64": 0}
    for p in probs:
        p["at"], p["elements"] = total[p["types"]], _elements(p["size"])
        total[p["types"]] += -(-p["elements"] // 64) * 64
    A = {t: _uniform(max(n, 1), t, gen) for t, n in total.items()}
    B = {t: _uniform(max(n, 1), t, gen) for t, n in total.items()}
    return probs, A, B


def _contraction_inputs(case, gen):
    ext = _ints(case["extents"])
    sizes = [[ext[l] for l in _ints(case[k])] for k in ("labels_a", "labels_b", "labels_c")]
    return sizes, [_uniform(_elements(s), case["types"], gen) for s in sizes]


def prepare(case, seed):
    gen = torch.Generator(device=_DEVICE).manual_seed(seed)
    if case["kind"] in ("call", "plan"):
        A, B, size, perm = _transposition_inputs(case, gen)
        alpha, beta = _scalars(case)
        state = dict(kind=case["kind"], A=A, B=B, size=size, perm=perm, alpha=alpha, beta=beta,
                     outer_a=_ints(case["outer_a"]), outer_b=_ints(case["outer_b"]))
        if case["kind"] == "plan":
            ta, tb = _PAIRS[case["types"]]
            plan = ttx.ttx_plan_create(ttx.CODE_OF[(_CODE[ta], _CODE[tb])], perm, size, state["outer_a"],
                                       state["outer_b"])
            state["plan"] = _Kept(plan, ttx.ttx_plan_destroy)
            ttx.ttx_plan_specialise(plan, beta == 0)
        return state
    if case["kind"] == "batch":
        probs, A, B = _batch_inputs(case, gen)
        batch = ttx.ttx_batch_create([
            ttx.make_problem(_CODE[p["types"]], p["perm"], p["size"], p["alpha"],
                             A[p["types"]][p["at"]:].data_ptr(), p["beta"], B[p["types"]][p["at"]:].data_ptr())
            for p in probs])
        return dict(kind="batch", batch=_Kept(batch, ttx.ttx_batch_destroy), A=A, B=B)
    sizes, (A, B, C) = _contraction_inputs(case, gen)
    plan = ttx.ttx_contraction_create(_CODE[case["types"]], _ints(case["labels_a"]), sizes[0],
                                      _ints(case["labels_b"]), sizes[1], _ints(case["labels_c"]), sizes[2])
    kept = _Kept(plan, ttx.ttx_contraction_destroy)
    workspace = torch.empty(ttx.ttx_contraction_describe(plan)["workspace_bytes"], dtype=torch.uint8, device=_DEVICE)
    return dict(kind="contraction", plan=kept, A=A, B=B, C=C, workspace=workspace, alpha=case["alpha"],
                beta=case["beta"])


def run(state):
    kind = state["kind"]
    if kind == "call":
        ttx.transpose(state["A"], state["B"], state["perm"], state["size"], state["alpha"], state["beta"],
                      state["outer_a"], state["outer_b"])
        return state["B"]
    if kind == "plan":
        A, B, alpha, beta = state["A"].data_ptr(), state["B"].data_ptr(), state["alpha"], state["beta"]
        if isinstance(alpha, complex):
            ttx.ttx_plan_execute_c(state["plan"].handle, alpha, A, beta, B, B, ttx.current_stream())
        else:
            ttx.ttx_plan_execute(state["plan"].handle, alpha, A, beta, B, ttx.current_stream())
        return state["B"]
    if kind == "batch":
        ttx.ttx_batch_execute(state["batch"].handle, ttx.current_stream())
        return state["B"]
    ttx.ttx_contraction_execute(state["plan"].handle, state["alpha"], state["A"].data_ptr(), state["B"].data_ptr(),
                                state["beta"], state["C"].data_ptr(), state["workspace"].data_ptr(),
                                ttx.current_stream())
    return state["C"]


def work(case):
    if case["kind"] in ("call", "plan"):
        ta, tb = _PAIRS[case["types"]]
        n = _elements(_ints(case["size"]))
        zero = _scalars(case)[1] == 0
        per = (1 if zero else 3) * (4 if tb in ("c32", "c64") else 1)
        return dict(bytes=n * (_BYTES[ta] + _BYTES[tb] * (1 if zero else 2)), flops=n * per)
    if case["kind"] == "batch":
        total = dict(bytes=0, flops=0)
        for p in _batch_problems(case):
            n, w = _elements(p["size"]), _BYTES[p["types"]]
            total["bytes"] += n * w * (2 if p["beta"] == 0 else 3)
            total["flops"] += n * (1 if p["beta"] == 0 else 3)
        return total
    ext, w = _ints(case["extents"]), _BYTES[case["types"]]
    a, b, c = (_elements([ext[l] for l in _ints(case[k])]) for k in ("labels_a", "labels_b", "labels_c"))
    k = _elements([ext[l] for l in set(_ints(case["labels_a"])) & set(_ints(case["labels_b"]))])
    return dict(bytes=w * (a + b + c * (1 if case["beta"] == 0 else 2)), flops=2 * c * k)


def _wide(x):
    return x.to(torch.complex128 if x.is_complex() else torch.float64)


def _rounded(v, dtype):
    """A scalar rounded to B's element type, as Eqn. 1 takes it."""
    return torch.tensor(v, dtype=_TORCH[dtype]).item()


def _exact_transposition(A, B, size, perm, alpha, beta, outer_a, outer_b):
    """Eqn. 1 in 64 bits on the flat column-major B (a new tensor)."""
    n = len(size)
    a = A.reshape((outer_a or size)[::-1])[tuple(slice(0, s) for s in size[::-1])]
    out = _wide(B).clone()
    sub_size = [size[k] for k in perm]
    b = out.view((outer_b or sub_size)[::-1])[tuple(slice(0, s) for s in sub_size[::-1])]
    # dimension j of the reversed view is index n - 1 - j
    moved = a.permute([n - 1 - perm[n - 1 - j] for j in range(n)])
    b.copy_(alpha * _wide(moved) + (beta * b if beta != 0 else 0))
    return out


def exact(case, seed):
    gen = torch.Generator(device=_DEVICE).manual_seed(seed)
    if case["kind"] in ("call", "plan"):
        A, B, size, perm = _transposition_inputs(case, gen)
        alpha, beta = (_rounded(v, _PAIRS[case["types"]][1]) for v in _scalars(case))
        A = A.to(torch.promote_types(B.dtype, torch.float32) if A.dtype != B.dtype else A.dtype)
        return _exact_transposition(A, B, size, perm, alpha, beta, _ints(case["outer_a"]), _ints(case["outer_b"]))
    if case["kind"] == "batch":
        probs, A, B = _batch_inputs(case, gen)
        out = {t: _wide(x).clone() for t, x in B.items()}
        for p in probs:
            t, at = p["types"], slice(p["at"], p["at"] + p["elements"])
            out[t][at] = _exact_transposition(A[t][at], B[t][at], list(p["size"]), list(p["perm"]),
                                              _rounded(p["alpha"], t), _rounded(p["beta"], t), None, None)
        return out
    sizes, (A, B, C) = _contraction_inputs(case, gen)
    la, lb, lc = (_ints(case[k]) for k in ("labels_a", "labels_b", "labels_c"))
    summed = [l for l in la if l in lb]
    # reversed shapes: the column-major tensors as torch's row-major ones
    a, b, c = (_wide(x).view(s[::-1]) for x, s in zip((A, B, C), sizes))
    prod = torch.tensordot(a, b, ([la[::-1].index(l) for l in summed], [lb[::-1].index(l) for l in summed]))
    left = [l for l in la[::-1] if l not in summed] + [l for l in lb[::-1] if l not in summed]
    prod = prod.permute([left.index(l) for l in lc[::-1]])
    return (case["alpha"] * prod + (case["beta"] * c if case["beta"] != 0 else 0)).reshape(-1)
