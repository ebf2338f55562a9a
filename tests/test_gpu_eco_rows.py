"""The zero-error scan where its division of work changes: one workgroup or several, trees of rows cut short by the end of
the tensor, more rows than wavefronts, an odd number of elements.  Counts against torch's, exact."""
import pytest
import torch

from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu
ROW, TREE = 128, 4 * 128


@pytest.mark.parametrize("n", [1, ROW - 1, ROW + 1, 16 * TREE - 1, 16 * TREE, 16 * TREE + 1, 17 * TREE + ROW + 3, 256 * 16 * ROW,
                               256 * 16 * TREE - ROW - 1, 256 * 16 * TREE + 5, 2 * 256 * 16 * TREE + 77])
def test_eco_scan_counts_at_the_edges_of_its_division(n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = (torch.randn(n, generator=g, device="cuda") * 2.0**20).to(torch.int64)
    s0 = torch.randint(-2**62, 2**62, (n,), generator=g, device="cuda", dtype=torch.int64)
    counts = torch.full((64,), -1, dtype=torch.int64, device="cuda")
    hb.hb_eco_scan(s0, x - s0, counts)
    d = x ^ (x >> 63)
    assert torch.equal(counts, torch.stack([((d >> b) & 1).sum() for b in range(64)]))
