"""Updates of a batch against a recording HIP runtime (no GPU): whatever the
new scalars, the launches find their tables, also where device memory has run
out since the batch was created."""
import pytest

import fake_hip

_BATCH = """
import random
import workloads
def batch(seed, betas):
    # a few uneven problems at made-up addresses; betas[i % len(betas)] each
    r, at, out = random.Random(seed), 1 << 40, []
    for i in range(r.choice([1, 2, 5])):
        n = r.randint(2, 4)
        size = [r.choice([3, 8, 17, 32, 60, 96, 200]) for _ in range(n)]
        perm = list(range(n))
        r.shuffle(perm)
        es = r.choice([4, 8])
        step = (workloads.elements(size) * es + 511) // 256 * 256
        out.append(ttx.make_problem(ttx.F32 if es == 4 else ttx.F64, perm, size, 1.5, at, betas[i % len(betas)], at + step))
        at += 2 * step
    return out
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake"))


def test_updates_allocate_nothing_and_keep_launches_sound(runtime):
    fake_hip.run(runtime, _BATCH + """
launched = 0
for seed in range(60):
    for before, after in (([0.0], [0.5]), ([0.5], [0.0]), ([0.0, 0.5], [0.5, 0.0])):
        fake.fake_reset()
        b = ttx.ttx_batch_create(batch(seed, before))
        ttx.ttx_batch_execute(b)
        fake.fake_fail_mallocs_after(0)
        for betas in (after, before, after):
            ttx.ttx_batch_update(b, batch(seed, betas))
            ttx.ttx_batch_execute(b)
            ttx.ttx_batch_execute_direct(b)
        ttx.ttx_batch_destroy(b)
        launched += sum("k_box_batch" in name for name, _, _ in launches())
        assert fake.fake_unsound() == 0, (seed, before, after)
assert launched > 500, launched
""")


def test_updates_choose_no_boxes_again(runtime):
    """A batch's shapes stay: each problem's boxes are chosen once per beta class."""
    fake_hip.run(runtime, _BATCH + """
for seed in range(12):
    q = batch(seed, [0.0])
    fake.fake_reset()
    b = ttx.ttx_batch_create(q)
    assert fake.fake_plans() == len(q), (fake.fake_plans(), len(q))
    ttx.ttx_batch_update(b, batch(seed, [0.0]))
    assert fake.fake_plans() == len(q), (fake.fake_plans(), len(q))
    for betas in ([0.5], [0.0], [-0.25], [0.0, 0.5]):
        ttx.ttx_batch_update(b, batch(seed, betas))
    assert fake.fake_plans() == 2 * len(q), (fake.fake_plans(), len(q))
    ttx.ttx_batch_destroy(b)
""")


def test_creation_costs_what_planning_costs(runtime):
    """The choice of boxes for 512 uneven problems takes about the host time of
    the heuristic configurations that it stands in for (ttx_batch_plan): best
    of 15 rounds each, in turn."""
    fake_hip.run(runtime, """
import ctypes, time
import workloads
from paper_1607_01249_amd import _ttx
at, problems = 1 << 40, []
for p in workloads.batched_problems():
    step = (workloads.elements(p["size"]) * p["dtype"].itemsize + 511) // 256 * 256
    problems.append(ttx.make_problem(ttx.F32 if p["dtype"].itemsize == 4 else ttx.F64, p["perm"], p["size"], p["alpha"],
                                     at, p["beta"], at + step))
    at += 2 * step
array, n, L = _ttx._problem_array(problems), len(problems), ttx.lib()
configs, tiles, batch = (ttx.Config * n)(), (ctypes.c_int64 * n)(), ctypes.c_void_p()
create = plan = 1e9
for _ in range(15):
    t0 = time.process_time()
    assert L.ttx_batch_create(ctypes.byref(batch), n, array) == 0
    t1 = time.process_time()
    assert L.ttx_batch_plan(n, array, configs, tiles) == 0
    t2 = time.process_time()
    L.ttx_batch_destroy(batch)
    create, plan = min(create, t1 - t0), min(plan, t2 - t1)
print("create %.2f ms, plan %.2f ms, %.2f" % (create * 1e3, plan * 1e3, create / plan))
assert create < 1.6 * plan, (create, plan)
""")
