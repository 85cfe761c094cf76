"""Box tiles (the per-call entry points) against the tile kernel of the
configuration that a plan describes, byte for byte, and against the oracle
(at most 1 ulp: the operation order is the same; gaps of B keep their values).
Shapes at the edges: cut indices with remainders (also shorter than a 16-byte
unit), runs that end inside a unit, runs cut by one index on both sides,
leading dimensions with an index that fills the box, LDS strides of powers of
two, one box, many boxes."""
import numpy as np
import pytest

import oracle
import paper_1607_01249_amd as ttx
import workloads
from gpu_util import (C32, C64, F32, F64, assert_parity, dtype_code, from_device, gpu_transpose, to_device)

pytestmark = pytest.mark.gpu

TYPES = [(F32, F32), (F64, F64), (C32, C32), (C64, C64), (F32, F64), (F64, F32), (C32, C64), (C64, C32)]
TYPE_IDS = ["s", "d", "c", "z", "sd", "ds", "cz", "zc"]
SHAPES = [   # perm, size, outer_a, outer_b
    ((1, 0), (65, 193), None, None), ((1, 0), (8, 4100), None, None), ((1, 0), (7, 4099), None, None),
    ((1, 0), (2, 5000), None, None), ((2, 1, 0), (129, 3, 130), None, None), ((2, 0, 1), (24, 20, 9), None, None),
    ((0, 2, 1), (63, 57, 5), None, None), ((0, 3, 2, 1), (5, 8, 21, 34), None, None),
    ((1, 0, 3, 2), (3, 13, 11, 257), None, None), ((5, 4, 3, 2, 1, 0), (5, 3, 7, 4, 6, 9), None, None),
    ((0, 1), (28, 900), (30, 900), (33, 901)), ((1, 0, 2), (70, 36, 9), (75, 40, 9), (37, 75, 12)),
    ((0, 2, 1), (9, 50, 40), (12, 52, 41), (11, 41, 51)), ((2, 1, 0), (1025, 2, 33), (1027, 2, 34), (34, 3, 1025)),
]


def _scalars(db, beta_zero):
    if db in (C32, C64):
        return complex(0.75, -1.25), (0j if beta_zero else complex(-0.5, 0.375))
    return 1.3, (0.0 if beta_zero else 0.7)


def _inputs(perm, size, da, db, outer_a, outer_b, seed):
    A = workloads.uniform(workloads.elements(outer_a or size), da, seed=300 + seed) * 3
    B = workloads.uniform(workloads.elements(outer_b or [size[p] for p in perm]), db, seed=700 + seed)
    return A, B


def _described(perm, size, da, db, outer_a, outer_b, beta_zero):
    plan = ttx.ttx_plan_create(dtype_code(da, db), perm, size, outer_a, outer_b)
    try:
        return ttx.ttx_plan_describe(plan)["config_raw"][int(beta_zero)]
    finally:
        ttx.ttx_plan_destroy(plan)


@pytest.mark.parametrize("beta_zero", [False, True], ids=["beta", "beta0"])
@pytest.mark.parametrize("types", TYPES, ids=TYPE_IDS)
def test_per_call_matches_tile_kernels_and_oracle(types, beta_zero):
    da, db = types
    alpha, beta = _scalars(db, beta_zero)
    for i, (perm, size, oa, ob) in enumerate(SHAPES):
        A, B = _inputs(perm, size, da, db, oa, ob, i)
        ref = B.copy()
        assert oracle.transpose(perm, size, alpha, A, beta, ref, oa, ob) == 0
        config = _described(perm, size, da, db, oa, ob, beta_zero)
        for pad_a, pad_b in ((0, 0), (1, 3)):
            got = gpu_transpose(perm, size, alpha, A, beta, B, oa, ob, pad_a, pad_b)
            tiles = gpu_transpose(perm, size, alpha, A, beta, B, oa, ob, pad_a, pad_b, plan_config=config)
            assert np.array_equal(got.view(np.uint8), tiles.view(np.uint8)), (perm, size, pad_a, "tile kernel")
            assert_parity(got, ref, False, (perm, size, pad_a))


@pytest.mark.parametrize("types", [TYPES[0], TYPES[3], TYPES[4], TYPES[7]], ids=["s", "z", "sd", "zc"])
def test_specialised_boxes_match_plans(types):
    """The box kernel compiled for a problem (its source names the box, and it
    takes pointers of any alignment) gives the bytes of the tile kernel."""
    da, db = types
    alpha, beta = _scalars(db, False)
    for i in (0, 3, 8, 9, 11):
        perm, size, oa, ob = SHAPES[i]
        plan = ttx.ttx_plan_create(dtype_code(da, db), perm, size, oa, ob)
        try:
            assert ttx.ttx_plan_specialise(plan, False)
            name = ttx.ttx_plan_kernel_name(plan, 0.5, 1 << 20, 3 << 20)
            assert name.startswith("ttx_jit_") and "_box" in name, name
            assert "ttx::BoxShape kHost" in ttx.ttx_plan_specialised_source(plan, False)
        finally:
            ttx.ttx_plan_destroy(plan)
        A, B = _inputs(perm, size, da, db, oa, ob, i)
        want = gpu_transpose(perm, size, alpha, A, beta, B, oa, ob,
                             plan_config=_described(perm, size, da, db, oa, ob, False))
        for pad_a, pad_b in ((0, 0), (1, 3)):
            got = gpu_transpose(perm, size, alpha, A, beta, B, oa, ob, pad_a, pad_b, specialise=True)
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (perm, size, pad_a)


@pytest.mark.parametrize("dtype,perm,size", [(F32, (2, 1, 0), (515, 33, 1024)), (F64, (1, 0), (96, 90000))],
                         ids=["rows_cut", "long_runs"])
def test_large_outputs_in_whole_lines(dtype, perm, size):
    """Outputs of 64 MiB and more in whole 128-byte lines (nontemporal stores),
    per call and specialised, and the same where B does not start on a line."""
    A, B = _inputs(perm, size, dtype, dtype, None, None, 60)
    want = gpu_transpose(perm, size, 1.3, A, 0.0, B, plan_config=_described(perm, size, dtype, dtype, None, None, True))
    for pad in (0, 1):
        for specialise in (False, True):
            got = gpu_transpose(perm, size, 1.3, A, 0.0, B, pad_b=pad, specialise=specialise)
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (pad, specialise)


@pytest.mark.parametrize("copies", [1, 7], ids=["few_boxes", "more_boxes"])
def test_batch_of_boxes_matches_plans(copies):
    """The launch over many problems (problems of one box and of many, flat
    ones, leading dimensions, pointers off 16-byte boundaries; chunks of one
    box and of several) gives each problem the bytes that a plan gives it."""
    shapes = [x for x in SHAPES for _ in range(copies)]
    shapes += [((0,), (5,), None, None), ((0, 1), (129, 77), None, None), ((1, 0), (3, 3), None, None)]
    keep, problems, want = [], [], []
    for i, (perm, size, oa, ob) in enumerate(shapes):
        dtype, beta, pad = (F32, F64)[i % 2], (0.0, 0.7, -0.25)[i % 3], i % 4
        A, B = _inputs(perm, size, dtype, dtype, oa, ob, i)
        want.append(gpu_transpose(perm, size, 1.3, A, beta, B, oa, ob, pad, pad,
                                  plan_config=_described(perm, size, dtype, dtype, oa, ob, beta == 0)))
        (dA, pa), (dB, pb) = to_device(A, pad), to_device(B, pad)
        keep.append((dA, dB, pad))
        problems.append(ttx.make_problem(dtype_code(dtype), perm, size, 1.3, pa, beta, pb, oa, ob))
    batch = ttx.ttx_batch_create(problems)
    try:
        ttx.ttx_batch_execute(batch, ttx.current_stream())
        for i, (_, dB, pad) in enumerate(keep):
            got = from_device(dB, pad)
            assert np.array_equal(got.view(np.uint8), want[i].view(np.uint8)), shapes[i]
    finally:
        ttx.ttx_batch_destroy(batch)


def test_values_that_are_not_numbers_pass_through():
    """beta = 0 reads nothing of B; infinities and NaN of A arrive unchanged
    with alpha = 1 (bit for bit)."""
    perm, size = (2, 1, 0), (67, 5, 70)
    A, B = _inputs(perm, size, F32, F32, None, None, 40)
    A[::97], A[5::89], B[:] = np.inf, np.nan, np.nan
    ref = B.copy()
    assert oracle.transpose(perm, size, 1.0, A, 0.0, ref) == 0
    assert_parity(gpu_transpose(perm, size, 1.0, A, 0.0, B), ref, True)


def test_on_a_stream_and_in_a_graph():
    """Launches only: captured once, replayed, the same bits each time."""
    import torch
    perm, size = (1, 0), (65, 193)
    A, B = _inputs(perm, size, F64, F64, None, None, 50)
    dA, pa = to_device(A)
    dB, pb = to_device(B)
    run = lambda: ttx.ttx_transpose(ttx.F64, 2, perm, size, None, None, 1.3, pa, 0.7, pb, ttx.current_stream())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            run()
    graph.replay()
    graph.replay()
    got = from_device(dB)
    expect = B.copy()
    for _ in range(3):
        expect = gpu_transpose(perm, size, 1.3, A, 0.7, expect)
    assert np.array_equal(got, expect)
