"""The double-double logarithm and arctangent (ddmath.hpp built for the host) at the steps of their
tables, against 50-digit mpmath."""
import ctypes
import os

import mpmath as mp
import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2208_02382_amd", "libpic_hostcheck.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="host check library not built")


@pytest.fixture(scope="module")
def lib():
    mp.mp.dps = 50
    return ctypes.CDLL(LIB)


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def test_dd_functions_at_the_table_steps(lib):
    """Arguments half way between two table entries and on them: the largest and the zero reduced
    argument, where the series' narrow terms weigh most."""
    k = np.arange(0, 1024)
    for half in (0.0, 0.5):
        c = (k + half) / 1024.0
        x = 1.0 + c
        a = np.stack([x, x * 1e-17], axis=1).copy()
        out = np.empty_like(a)
        lib.pic_hostcheck_dd(0, len(x), _p(a), _p(out))
        for i in range(1, len(x), 3):
            ref = mp.log(mp.mpf(a[i, 0]) + mp.mpf(a[i, 1]))
            assert abs((mp.mpf(out[i, 0]) + mp.mpf(out[i, 1]) - ref) / ref) < 1e-30
        q = np.full(len(c), 0.75)
        b = np.stack([c * q, c * 1e-18, q, q * 1e-17], axis=1).copy()
        o2 = np.empty((len(c), 2))
        lib.pic_hostcheck_dd_atan2(len(c), _p(b), _p(o2))
        for i in range(1, len(c), 3):
            ref = mp.atan((mp.mpf(b[i, 0]) + mp.mpf(b[i, 1])) / (mp.mpf(b[i, 2]) + mp.mpf(b[i, 3])))
            assert abs((mp.mpf(o2[i, 0]) + mp.mpf(o2[i, 1]) - ref) / ref) < 1e-30
