"""GPU parity of the direct contraction kernels at the edges of their tiles
(64 or 128 rows; 16, 32, 64 or 80 columns; steps of 8 to 32 contracted
values), of their splits of the sum and of the forms of the operands' runs.

Integer-valued operands keep every product and partial sum exact in both
precisions (|sum| <= 16 * k < 2^24), whatever the order of the sum, so that
the results have to equal the oracle bit for bit."""
import numpy as np
import pytest

import paper_1607_01249_amd as ttx
from gpu_util import F32, F64, dtype_code, from_device, to_device
from oracle import tensor_contract as tc

pytestmark = pytest.mark.gpu

# (labels_a, labels_b, labels_c, extents): the operands' and C's stride-1
# labels in every role, runs that are whole 16-byte units and runs that are not
FORMS = [
    ((0, 2), (2, 1), (0, 1)),                # A along rows, B along the sum
    ((2, 0), (1, 2), (0, 1)),                # A along the sum, B along columns
    ((0, 2), (2, 1), (1, 0)),                # B holds C's stride-1 label
    ((3, 0, 2), (2, 3, 1), (0, 1)),          # both along the sum, over different labels
    ((4, 2, 0), (1, 2), (0, 4, 1)),          # A's run is not C's
    ((4, 2, 0), (5, 2, 1), (0, 1, 4, 5)),    # nor B's; C's runs go on through the columns
    ((0, 2, 4), (2, 1), (0, 1, 4)),          # C's runs are rows, then columns
]


def _extents(m, n, k):
    # labels 0, 1, 2 are the rows, the columns and the sum; 3, 4, 5 join them
    return {0: m, 1: n, 2: k, 3: 5, 4: 6, 5: 4}


def _check(la, lb, lc, ext, dtype, alpha, beta, seed):
    import torch
    sizes = [tuple(ext[l] for l in lab) for lab in (la, lb, lc)]
    rng = np.random.default_rng(seed)
    A, B, C = (rng.integers(-4, 5, size=int(np.prod(s, dtype=np.int64))).astype(dtype) for s in sizes)
    plan = ttx.ttx_contraction_create(dtype_code(dtype), la, sizes[0], lb, sizes[1], lc, sizes[2])
    try:
        ws = torch.full((ttx.ttx_contraction_describe(plan)["workspace_bytes"] // 4 + 1,), float("nan"),
                        dtype=torch.float32, device="cuda")
        (dA, pa), (dB, pb), (dC, pc) = to_device(A), to_device(B), to_device(C)
        print(la, lb, lc, ext, dtype, flush=True)
        ttx.ttx_contraction_execute(plan, alpha, pa, pb, beta, pc, ws.data_ptr(), ttx.current_stream())
        got = from_device(dC)
    finally:
        ttx.ttx_contraction_destroy(plan)
    want = tc.contract(la, A, sizes[0], lb, B, sizes[1], lc, sizes[2], alpha, beta, C, out_dtype=dtype)
    assert np.array_equal(got, want), (la, lb, lc, ext, np.flatnonzero(got != want)[:8])


@pytest.mark.parametrize("form", FORMS, ids=lambda f: "%s_%s_%s" % tuple("".join(map(str, x)) for x in f))
@pytest.mark.parametrize("dtype", [F32, F64], ids=["f32", "f64"])
def test_tile_edges(form, dtype):
    # k (times 5 where label 3 is summed too): one step and its edges, several steps, the table of 256 k values
    for i, (m, n, k) in enumerate([(64, 64, 16), (65, 17, 33), (63, 80, 7), (24, 16, 8), (128, 81, 1), (7, 9, 257),
                                   (130, 33, 64), (1, 1, 3), (16, 1, 40), (1, 31, 31)]):
        _check(*form, _extents(m, n, k), dtype, 1.0 if i % 2 else -0.5, 0.0 if i % 3 == 0 else 2.0, 40 + i)


@pytest.mark.parametrize("dtype", [F32, F64], ids=["f32", "f64"])
def test_split_sums(dtype):
    """Small results of long sums: the sum is cut over workgroups, the partial sums lie in the workspace."""
    for form, (m, n, k) in [(FORMS[0], (96, 64, 2048)), (FORMS[1], (33, 33, 1999)), (FORMS[3], (40, 20, 700)),
                            (FORMS[4], (9, 5, 3001)), (((0,), (0,), ()), (5000, 1, 1))]:
        _check(*form, _extents(m, n, k), dtype, 0.5, 2.0, 7)


@pytest.mark.parametrize("dtype,e,k", [(F32, 17, 16), (F32, 18, 5), (F64, 19, 8)])
def test_many_tiles_of_a_short_sum(dtype, e, k):
    """Large results of short sums (97 to 376 MB): the operands are packed into whole tiles in the workspace."""
    ext = dict.fromkeys(range(6), e)
    ext[6] = k
    for beta in (0.0, 1.0):
        _check((2, 6, 0, 4), (5, 3, 6, 1), (0, 1, 2, 3, 4, 5), ext, dtype, 1.0, beta, 3)
