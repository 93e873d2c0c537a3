"""The float32 butterflies of the register transforms (fft_reg.hpp built for the host) give impulses
of many amplitudes their roots without a bias: a rounded root, met in every line of every pass, scales
the field, where the roundings of the values average out.

Bar: a component passes at most five roundings to nearest (nested radices) of values below 2, each
uniform within 2^-24, of standard deviation 7.7e-8 together; the mean over 2^16 amplitudes has 3e-10,
and 2e-9 is asked.  A root's own rounding is up to 3e-8 (1.2e-8 for sqrt(1/2), 1.6e-8
for sqrt(3)/2)."""
import ctypes
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2208_02382_amd", "libpic_hostcheck.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="host check library not built")


@pytest.mark.parametrize("radix", [2, 3, 4, 6, 8, 9, 12, 16])
@pytest.mark.parametrize("sign", [-1, 1])
def test_float32_roots_have_no_bias(radix, sign):
    lib = ctypes.CDLL(LIB)
    m = 1 << 16
    a = np.random.default_rng(radix).uniform(1.0, 2.0, m).astype(np.float32)
    for j in range(radix):
        v = np.zeros((m, radix), dtype=np.complex64)
        v[:, j] = a
        lib.pic_hostcheck_dft(radix, sign, m, v.ctypes.data_as(ctypes.c_void_p))
        root = np.exp(sign * 2j * np.pi * j * np.arange(radix) / radix)
        bias = (v.astype(np.complex128) / a[:, None].astype(np.float64) - root).mean(axis=0)
        assert max(np.abs(bias.real).max(), np.abs(bias.imag).max()) < 2e-9
