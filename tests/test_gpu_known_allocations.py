"""The checks of a call ask for an allocation once: a buffer that runs over the end of an allocation, or of the GPU's memory at
all, is refused whether its allocation is new to the call or known from a buffer before."""
import ctypes

import pytest
import torch

from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu
MIB = 1 << 20


def _status(s0, s1, o0, o1, n):
    return hb.raw("hb_relu", s0, s1, n, 12, 20, 5, o0, o1, None, None)


def test_buffers_of_one_allocation_and_over_its_end():
    big = torch.zeros(64 * MIB // 8, dtype=torch.int64, device="cuda")       # an allocation of its own
    n, base, end = 1000, big.data_ptr(), big.data_ptr() + 64 * MIB
    at = [base + i * 8 * n for i in range(4)]
    assert _status(*at, n) == hb.HB_OK
    assert _status(at[0], at[1], at[2], end - 8 * n, n) == hb.HB_OK          # the last n words of it
    for i in range(4):                                                       # one word over the end, in every position
        over = list(at)
        over[i] = end - 8 * n + 8
        assert _status(*over, n) == hb.HB_EINVAL
    host = torch.zeros(n, dtype=torch.int64)
    for i in range(4):
        assert _status(*(at[:i] + [host.data_ptr()] + at[i + 1:]), n) == hb.HB_EINVAL
    torch.cuda.synchronize()


def test_a_set_of_more_allocations_than_are_kept():
    n = 1000
    bufs = [torch.zeros(32 * MIB // 8, dtype=torch.int64, device="cuda") for _ in range(20)]
    items = [[b[i * n:(i + 1) * n] for i in range(4)] + [12, 20, 3] for b in bufs]
    arr = hb.make_batch(items)
    assert hb.raw("hb_relu_batch", arr, len(items), None, None) == hb.HB_OK
    arr[19].out1 = bufs[0].data_ptr() + 32 * MIB - 8 * n + 8                 # known at first, dropped since
    assert hb.raw("hb_relu_batch", arr, len(items), None, None) == hb.HB_EINVAL
    arr[19].out1 = ctypes.c_void_p(bufs[19].data_ptr() + 32 * MIB - 8 * n + 8)
    assert hb.raw("hb_relu_batch", arr, len(items), None, None) == hb.HB_EINVAL
    torch.cuda.synchronize()
