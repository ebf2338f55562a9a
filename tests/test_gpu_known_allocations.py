"""The checks of a call ask for an allocation once: a buffer that runs over the end of an allocation, or of the GPU's memory at
all, is refused whether its allocation is new to the call or known from a buffer before.  The allocations come from the HIP
runtime itself, so that their ends are known (a tensor may be a piece of a larger cached block)."""
import ctypes

import pytest
import torch

from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.fixture
def allocate():
    torch.cuda.init()
    torch.zeros(1, device="cuda")
    hip = ctypes.CDLL(hb.LIBRARY)                   # its symbols include those of the runtime that the library is linked with
    hip.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    hip.hipFree.argtypes = [ctypes.c_void_p]
    taken = []

    def take(size):
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), size) == 0
        taken.append(p.value)
        return p.value

    yield take
    torch.cuda.synchronize()
    for p in taken:
        assert hip.hipFree(p) == 0


def _status(s0, s1, o0, o1, n):
    return hb.raw("hb_relu", s0, s1, n, 12, 20, 5, o0, o1, None, None)


def test_buffers_of_one_allocation_and_over_its_end(allocate):
    n, size = 1000, 64 * MIB
    base = allocate(size)
    end = base + size
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


def test_a_set_of_more_allocations_than_are_kept(allocate):
    n, size = 1000, 4 * MIB
    bases = [allocate(size) for _ in range(20)]
    arr = (hb.hb_tensor * len(bases))()
    for d, base in zip(arr, bases):
        d.share0, d.share1, d.out0, d.out1 = (base + i * 8 * n for i in range(4))
        d.n, d.k, d.m, d.seed = n, 12, 20, 3
    assert hb.raw("hb_relu_batch", arr, len(bases), None, None) == hb.HB_OK
    arr[19].out1 = bases[0] + size - 8 * n + 8                               # known at first, dropped since
    assert hb.raw("hb_relu_batch", arr, len(bases), None, None) == hb.HB_EINVAL
    arr[19].out1 = bases[19] + size - 8 * n + 8
    assert hb.raw("hb_relu_batch", arr, len(bases), None, None) == hb.HB_EINVAL
