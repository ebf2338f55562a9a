"""Three and four parties where the kernels draw dealer words in step: around the lines where that form begins, its quarters of a
tile, one thread per group, and outputs that are inputs (the shares of four parties at w = 4 are read a second time).  Bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu

SEED = 0x2309048750000056
DEV = "cuda"


def _check(parties, w, n, in_place=False):
    rng = np.random.default_rng(1000 * parties + 10 * w + n)
    k = int(rng.integers(0, 64 - w + 1))
    m, off = k + w, n % 2
    host = [rng.integers(0, 1 << 64, n + off, dtype=np.uint64).view(np.int64) for _ in range(parties)]
    s = [h[off:] for h in host]
    for call, what in ((hb.hb_relu_mp, oracle.WHAT_RELU), (hb.hb_drelu_mp, oracle.WHAT_DRELU)):
        d = [torch.from_numpy(h).to(DEV)[off:] for h in host]
        outs, _ = call(d, k, m, SEED, d[1:] + d[:1] if in_place else None)      # party q's result over party q + 1's share
        for g, r in zip(outs, oracle.mp_evaluate(s, k, m, SEED, what, threads=8)):
            assert np.array_equal(g.cpu().numpy(), r), (parties, w, n, call.__name__)


@pytest.mark.parametrize("parties", [3, 4])
@pytest.mark.parametrize("w", [4, 5, 8])
def test_quarters_of_a_tile(parties, w):
    per = 64 * min(64 // w, 64 // parties)
    for tiles in (258, 1025, 1282, 2050):
        _check(parties, w, tiles * per - 5)


@pytest.mark.parametrize("parties", [3, 4])
def test_one_bit_in_its_third_and_fourth_round(parties):
    per = 32 * (64 // parties)
    for tiles in (2048, 2049, 4096, 4097):
        _check(parties, 1, tiles * per - 5)


@pytest.mark.parametrize("parties", [3, 4])
@pytest.mark.parametrize("w", [33, 34, 64])
def test_one_thread_per_group(parties, w):
    for n in (65536, 65537):
        _check(parties, w, n)


@pytest.mark.parametrize("tiles", [3, 1600])
def test_results_over_shares(tiles):
    _check(4, 4, tiles * 1024 - 5, in_place=True)
