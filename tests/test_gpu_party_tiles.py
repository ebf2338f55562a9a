"""The party-faithful kernel at the edges of its tiles: a wavefront takes 32 groups, so a tile may end inside a 64-bit
word of the B2A message (odd L), inside a chunk of 64 elements of the multiply message, or before either.  Shares and
every wire word against the oracle's transcript, bit for bit, both dealer layouts; the workspace starts as all ones, so
a wire word that was not written shows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dealer", [hb.HB_DEALER_PER_GATE, hb.HB_DEALER_SHARED_MASK])
@pytest.mark.parametrize("k,m", [(0, 64), (3, 36), (5, 26), (1, 8), (12, 20), (4, 7), (9, 10), (8, 14)])
def test_party_kernel_at_tile_edges(k, m, dealer):
    L = min(64 // (m - k), 32)
    tile = 32 * L
    rng = np.random.default_rng(1000 * k + m)
    for n in sorted({tile - 1, tile, tile + 1, 2 * tile, 3 * tile, 3 * tile + L, 5 * tile - L + 1, 4 * tile + 32, 7 * tile}):
        s0, s1 = (rng.integers(0, 1 << 64, n, dtype=np.uint64).view(np.int64) for _ in range(2))
        seed = 0x2309048750000001 + n
        ws = torch.full((hb.hb_party_workspace_bytes_ex(n, k, m, dealer),), 255, dtype=torch.uint8, device=DEV)
        o0, o1, w0, w1, _ = hb.hb_relu_party_ex(torch.from_numpy(s0).to(DEV), torch.from_numpy(s1).to(DEV), k, m, seed, dealer,
                                                workspace=ws)
        e0, e1, _ = oracle.relu(s0, s1, k, m, seed, variant=dealer)
        x0, x1 = oracle.relu_wire(s0, s1, k, m, seed, variant=dealer)
        assert np.array_equal(o0.cpu().numpy(), e0) and np.array_equal(o1.cpu().numpy(), e1), (k, m, n)
        assert np.array_equal(w0.cpu().numpy().view(np.uint64), x0), (k, m, n)
        assert np.array_equal(w1.cpu().numpy().view(np.uint64), x1), (k, m, n)
