"""Launches of contractions whose tiles do not fit one grid (2^32 work items
and more are refused): several launches cover every workgroup once."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake"))


@pytest.mark.parametrize("dtype", ["F32", "F64"])
@pytest.mark.parametrize("m,n,k", [(2, 1 << 30, 1), (5, 1300000000, 2), (1 << 31, 1, 1), (1 << 30, 2, 40), (64, 64, 64)])
def test_every_launch_is_accepted(runtime, dtype, m, n, k):
    fake_hip.run(runtime, """
m, n, k = %d, %d, %d
es = 4 if "%s" == "F32" else 8
plan = ttx.ttx_contraction_create(ttx.%s, (0, 2), (m, k), (2, 1), (k, n), (0, 1), (m, n))
at, ptr = 1 << 41, []
for nbytes in (m * k * es, k * n * es, m * n * es, ttx.ttx_contraction_describe(plan)["workspace_bytes"]):
    ptr.append(at)
    at += nbytes + 256
ttx.ttx_contraction_execute(plan, 1.0, ptr[0], ptr[1], 0.5, ptr[2], ptr[3])
assert fake.fake_unsound() == 0, launches()
by_kernel = {}
for name, grid, first in launches():
    by_kernel.setdefault(name, []).append((first, grid))
assert any("k_contract" in name for name in by_kernel), by_kernel
assert k != 1 or m * n < 1 << 31 or any(len(v) > 1 for v in by_kernel.values()), by_kernel
for ranges in by_kernel.values():      # one after the other, from 0 on
    assert all(first == sum(g for _, g in ranges[:i]) for i, (first, _) in enumerate(ranges)), ranges
""" % (m, n, k, dtype, dtype))
