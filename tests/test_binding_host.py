"""The per-call binding passes its integer arrays as packed bytes: the same
bytes as ctypes arrays for everything that int() takes."""
import ctypes

import numpy as np
import pytest

from paper_1607_01249_amd import _ttx


@pytest.mark.parametrize("fmt,ctype", [("i", ctypes.c_int), ("q", ctypes.c_int64)])
@pytest.mark.parametrize("vals", [[3, 2, 1], (0,), np.array([5, 6, 7]), [2.0, 3], [np.int64(4), True], list(range(20)),
                                  [2 ** 40, -1], ["7"]], ids=str)
def test_packed_arrays_equal_ctypes_arrays(vals, fmt, ctype):
    assert _ttx._packed(vals, fmt) == bytes(_ttx._ints(vals, ctype))


def test_nothing_and_no_integers():
    assert _ttx._packed(None, "q") is None
    with pytest.raises(ValueError):
        _ttx._packed(["x"], "i")
    with pytest.raises(TypeError):
        _ttx._packed([None], "q")
