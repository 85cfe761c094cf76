"""Size-specialised box kernels of large outputs in whole lines (nontemporal
stores where B starts on a 128-byte line): a B that starts elsewhere runs the
plan's compiled kernel too, with the same bytes."""
import numpy as np
import pytest

import paper_1607_01249_amd as ttx
import workloads
from gpu_util import F32, F64, dtype_code, from_device, gpu_transpose, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,perm,size", [(F32, (2, 1, 0), (515, 33, 1024)), (F64, (1, 0), (96, 90000))],
                         ids=["rows_cut", "long_runs"])
def test_compiled_kernel_for_every_alignment(dtype, perm, size):
    A = workloads.uniform(workloads.elements(size), dtype, seed=5) * 3
    plan = ttx.ttx_plan_create(dtype_code(dtype), perm, size)
    try:
        want = gpu_transpose(perm, size, 1.3, A, 0.0, A,
                             plan_config=ttx.ttx_plan_describe(plan)["config_raw"][1])
        assert ttx.ttx_plan_specialise(plan, True)
        dA, pa = to_device(A)
        for pad in (0, 16 // dtype.itemsize, 64 // dtype.itemsize, 1):
            dB, pb = to_device(np.zeros_like(A), pad)
            name = ttx.ttx_plan_kernel_name(plan, 0.0, pa, pb)
            assert name.startswith("ttx_jit_") and "_b0_box" in name, (pad, name)
            assert name.endswith("_off_line") == (pb % 128 != 0), (pad, name)
            ttx.ttx_plan_execute(plan, 1.3, pa, 0.0, pb, ttx.current_stream())
            assert np.array_equal(from_device(dB, pad).view(np.uint8), want.view(np.uint8)), pad
    finally:
        ttx.ttx_plan_destroy(plan)
