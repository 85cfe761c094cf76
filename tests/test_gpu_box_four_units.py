"""Boxes of four units a thread, per call and specialised, in every type and
beta class: the bytes of the tile kernel of the configuration that a plan
describes, and the oracle's values (at most 1 ulp)."""
import numpy as np
import pytest

import oracle
import paper_1607_01249_amd as ttx
from gpu_util import C64, F32, assert_parity, dtype_code, gpu_transpose
from test_gpu_box import TYPES, TYPE_IDS, _described, _inputs, _scalars

pytestmark = pytest.mark.gpu


def _check(perm, size, types, beta_zero, pads, seed):
    da, db = types
    alpha, beta = _scalars(db, beta_zero)
    plan = ttx.ttx_plan_create(dtype_code(da, db), perm, size)
    try:
        assert ttx.ttx_plan_specialise(plan, beta_zero)
        assert ", 4, " in ttx.ttx_plan_specialised_source(plan, beta_zero)   # the units a thread
    finally:
        ttx.ttx_plan_destroy(plan)
    A, B = _inputs(perm, size, da, db, None, None, seed)
    want = gpu_transpose(perm, size, alpha, A, beta, B, plan_config=_described(perm, size, da, db, None, None, beta_zero))
    ref = B.copy()
    assert oracle.transpose(perm, size, alpha, A, beta, ref) == 0
    assert_parity(want, ref, False, (perm, size))
    for pad in pads:
        for specialise in (False, True):
            got = gpu_transpose(perm, size, alpha, A, beta, B, pad_a=pad, pad_b=pad, specialise=specialise)
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (pad, specialise)


@pytest.mark.parametrize("beta_zero", [False, True], ids=["beta", "beta0"])
@pytest.mark.parametrize("types", TYPES, ids=TYPE_IDS)
def test_four_units_match_tile_kernels(types, beta_zero):
    perm, size = ((1, 0, 3, 2), (20, 26, 18, 25)) if types == (C64, C64) else ((3, 1, 2, 0), (22, 25, 25, 25))
    _check(perm, size, types, beta_zero, (0, 1), 70)


def test_four_units_with_nontemporal_stores():
    """79 MB in whole lines, and with B off a line."""
    _check((1, 0, 3, 2), (32, 70, 160, 55), (F32, F32), True, (0, 1), 71)
