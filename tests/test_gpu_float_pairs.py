"""hb_share_f32 and hb_reveal_f32, a pair of elements per lane: odd sizes, edges of a workgroup, buffers that are only
element-aligned.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [1, 2, 3, 511, 512, 513, 1023, 100001])
@pytest.mark.parametrize("float_offset", [0, 1])
@pytest.mark.parametrize("share_offset", [0, 1])
def test_share_and_reveal(n, float_offset, share_offset):
    x = (np.random.default_rng(n).standard_normal(n) * 300).astype(np.float32)
    d = torch.zeros(n + 2, device=DEV)[float_offset:float_offset + n]
    d.copy_(torch.from_numpy(x))
    whole = [torch.full((n + 3,), -7, dtype=torch.int64, device=DEV) for _ in range(2)]
    s = [t[share_offset:share_offset + n] for t in whole]
    hb.hb_share_f32(d, 99, s[0], s[1])
    e = oracle.share_f32(x, 99)
    for t, q, ref in zip(whole, s, e):
        assert np.array_equal(q.cpu().numpy(), ref)
        assert (t[:share_offset] == -7).all() and (t[share_offset + n:] == -7).all()
    y = torch.full((n + 2,), -7.0, device=DEV)
    hb.hb_reveal_f32(s[0], s[1], y[float_offset:float_offset + n])
    assert np.array_equal(y[float_offset:float_offset + n].cpu().numpy(), oracle.reveal_f32(*e))
    assert (y[:float_offset] == -7).all() and (y[float_offset + n:] == -7).all()
