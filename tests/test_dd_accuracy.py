"""The double-double logarithm, arctangent, square root and quotient of the integrated Green's function
(ddmath.hpp built for the host) against 60-digit mpmath, within their roundings' bounds."""
import ctypes
import os

import numpy as np
import pytest

import dd_accuracy

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2208_02382_amd", "libpic_hostcheck.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="host check library not built")


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("name", sorted(dd_accuracy.arguments()))
def test_operations_are_within_their_roundings(name):
    lib = ctypes.CDLL(LIB)
    fn, arg = dd_accuracy.arguments()[name]
    out = np.zeros((len(arg), 2))
    if fn in (0, 2):
        one = np.ascontiguousarray(arg[:, :2])
        lib.pic_hostcheck_dd(fn, len(arg), _p(one), _p(out))
    else:
        f = lib.pic_hostcheck_dd_atan2 if fn == 1 else lib.pic_hostcheck_dd_div
        f(len(arg), _p(arg), _p(out))
    assert dd_accuracy.worst(fn, arg, out) < 1.0
