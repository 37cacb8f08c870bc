"""The shared square roots (csrc/roots.h) against sqrtf, bit for bit: every float, and waves
in which one lane's zero, denormal, small, infinite or NaN value sends the others' ordinary
ones down the other path.  The localiser compares an intensity from sqrtf with a threshold
from these roots, so they have to be the same."""
import ctypes
import os

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "_build", "libroots_check.so")


@pytest.fixture(scope="module")
def check():
    import torch
    assert os.path.exists(LIB), "run __graft_entry__.build()"
    fn = ctypes.CDLL(LIB).roots_check
    fn.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int, ctypes.c_uint32,
                   ctypes.c_void_p, ctypes.c_void_p]
    fn.restype = ctypes.c_int

    def run(first, threads, stride=0, odd=None):
        bad = torch.zeros(1, dtype=torch.int64, device="cuda")
        st = fn(first, threads, stride, odd is not None, odd or 0, bad.data_ptr(),
                torch.cuda.current_stream().cuda_stream)
        assert st == 0
        return int(bad.item())

    return run


def test_every_float(check):
    # runs of neighbours, eight a thread
    for q in range(256):
        assert check(q << 24, 1 << 21) == 0, f"bit patterns from {q << 24:#x}"
    say("[roots] 2^32 floats equal")


def test_spread_values(check):
    # a thread's eight values far apart, both sides of 2^-96 in one wave among them
    for first in (0, 0x0f7ff000, 0x0f800000, 0x3f800000, 0x7f7f0000):
        assert check(first, 1 << 20, stride=1 << 28) == 0
        assert check(first, 1 << 20, stride=(1 << 23) + 1) == 0


@pytest.mark.parametrize("odd", [0x00000000, 0x80000000, 0x00000001, 0x007fffff, 0x0f7fffff, 0x7f800000, 0x7fc00000,
                                 0xbf800000])
def test_mixed_waves(check, odd):
    for first in (0x0f800000, 0x1f000000, 0x3f000000, 0x5f000000, 0x7f000000):
        assert check(first, 1 << 20, odd=odd) == 0
