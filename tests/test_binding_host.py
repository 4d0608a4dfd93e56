"""Array arguments of the Python binding: the address of a numpy array's data,
whatever its layout; other buffers, whose element type the library would not
know, are refused."""

import array
import ctypes

import numpy as np
import pytest

import paper_0902_4463_amd as g6


def test_addresses_of_arrays():
    a = np.arange(12.0).reshape(4, 3)
    ro = a.copy()
    ro.flags.writeable = False
    for q in (a, a[::2], a.T, ro, np.zeros(0), np.zeros((), dtype=np.int32)):
        assert g6._pd(q) == q.ctypes.data
    assert g6._pd(None) is None


@pytest.mark.parametrize("bad", [bytearray(64), memoryview(bytearray(64)), array.array("f", [0.0] * 8),
                                 (ctypes.c_float * 8)(), [0.0], 5])
def test_other_buffers_are_refused(bad):
    with pytest.raises(AttributeError):
        g6._pd(bad)
