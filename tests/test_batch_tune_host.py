"""What ttx_batch_tune makes of given times (no GPU): a problem in box tiles
takes whichever configuration is clearly faster than its boxes, the heuristic
one too, and its boxes are timed with the kernel variant that the batch runs."""
import pytest

import fake_hip

_TUNE = """
def tuned(first, rest, boxes, size=(96, 64, 32), beta=0.0):
    fake.fake_reset()
    fake.fake_times(1, (ctypes.c_double * 1)(first), ctypes.c_double(rest), ctypes.c_double(boxes))
    step = 1 << 38
    b = ttx.ttx_batch_create([ttx.make_problem(ttx.F32, (2, 1, 0), size, 1.5, step, beta, 2 * step)])
    ttx.ttx_batch_execute(b)
    assert "k_box_batch" in launches()[-1][0]
    ttx.ttx_batch_tune(b)
    timed = launches()
    ttx.ttx_batch_execute(b)
    ttx.ttx_batch_execute_direct(b)
    after = [name for name, _, _ in launches()[len(timed):]]
    ttx.ttx_batch_destroy(b)
    assert fake.fake_unsound() == 0
    return after, [name for name, _, _ in timed]
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake"))


@pytest.mark.parametrize("first,rest,boxes,kernel", [(1, 5, 5, "k_batch"), (5, 1, 5, "k_batch"), (5, 5, 1, "k_box_batch"),
                                                     (4.9, 5, 5, "k_box_batch")])
def test_the_clearly_faster_one_runs(runtime, first, rest, boxes, kernel):
    fake_hip.run(runtime, _TUNE + """
after, _ = tuned(%r, %r, %r)
assert len(after) == 2 and all(%r in name for name in after), after
""" % (first, rest, boxes, kernel))


def test_boxes_are_timed_with_plain_stores(runtime):
    fake_hip.run(runtime, _TUNE + """
_, timed = tuned(5, 5, 1, size=(512, 64, 1024))
names = [n for n in timed if "5k_box" in n]
assert names and not any("Lb1EEEv" in n for n in names), names   # the last parameter: nontemporal stores
""")
