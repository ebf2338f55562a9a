"""Launches whose kernels draw dealer words in step (the forms with RUNS), where other tests do not reach them: sizes at the
lines where they begin, their quarters of a tile, and the widths of one thread per group.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu

SEED = 0x2309048750000055
DEV = "cuda"
LAYOUTS = (hb.HB_DEALER_PER_GATE, hb.HB_DEALER_SHARED_MASK)


def _check(w, n, seed):
    rng = np.random.default_rng(seed)
    k = int(rng.integers(0, 64 - w + 1))
    m, off = k + w, n % 2                                      # odd sizes on buffers that are only 8-byte aligned
    host = [rng.integers(0, 1 << 64, n + off, dtype=np.uint64).view(np.int64) for _ in range(2)]
    d = [torch.from_numpy(h).to(DEV)[off:] for h in host]
    s = [h[off:] for h in host]

    def same(what, got, ref):
        assert all(np.array_equal(g.cpu().numpy(), r) for g, r in zip(got, ref)), (what, w, n)

    for layout in LAYOUTS:
        for call, ref in ((hb.hb_relu_ex, oracle.relu), (hb.hb_drelu_ex, oracle.drelu)):
            same((call.__name__, layout), call(d[0], d[1], k, m, SEED, layout)[:2], ref(s[0], s[1], k, m, SEED, variant=layout, threads=8)[:2])
    same("sign", hb.hb_sign_shares(d[0], d[1], k, m, SEED)[:2], oracle.evaluate(s[0], s[1], k, m, SEED, oracle.WHAT_SIGN, threads=8))
    x = (rng.standard_normal(n) * 2).astype(np.float32)
    y = hb.hb_sim_relu_f32(torch.from_numpy(x).to(DEV), k, m, SEED, 5)
    same("simulator", [y], [oracle.sim_relu_f32(x, k, m, SEED, 5, threads=8)])


@pytest.mark.parametrize("w", range(4, 13))
def test_quarters_of_a_tile(w):
    per = 64 * (64 // w)
    for tiles in (258, 1025, 1346, 2051):                      # all by quarters; around the line; three tiles after two full rounds
        _check(w, tiles * per - 5, 100 * w + tiles)


@pytest.mark.parametrize("w", [33, 34, 48, 63, 64])
def test_one_thread_per_group(w):
    for n in (65536, 65537, 70001):                            # 256 workgroups are the most without
        _check(w, n, w + n)
