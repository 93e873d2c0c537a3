"""The double-double operations of the integrated Green's function on the device, whose reciprocals
start from the hardware's, at the bars of the host build's test."""
import ctypes
import os

import pytest
import torch

import dd_accuracy

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2208_02382_amd", "libpic_devcheck.so")


@pytest.mark.parametrize("name", sorted(dd_accuracy.arguments()))
def test_operations_are_within_their_roundings(name):
    lib = ctypes.CDLL(LIB)
    fn, arg = dd_accuracy.arguments()[name]
    d_in = torch.from_numpy(arg).cuda()
    d_out = torch.zeros((len(arg), 2), dtype=torch.float64, device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.pic_devcheck_dd(fn, len(arg), ctypes.c_void_p(d_in.data_ptr()),
                               ctypes.c_void_p(d_out.data_ptr()), stream) == 0
    assert dd_accuracy.worst(fn, arg, d_out.cpu().numpy()) < 1.0
