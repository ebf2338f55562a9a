"""Launches whose last tiles are shared out by quarters: sizes around the rule's lines, bit for bit against the oracle.

A tile has 64 groups.  Up to 256 to 1280 tiles, by width and operation, every tile goes to a workgroup by quarters, above that what is
left after the last 1024 whole ones if it is at most 256 or 512; the tensors here end one element short of a tile or five elements into one (whose
other quarters are then empty), and the batched call has the line between whole and shared-out tiles inside a tensor.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_04875_amd import hb, workloads

pytestmark = pytest.mark.gpu

SEED = 0x2309048750000077
DEV = "cuda"


def _shares(n, seed):
    _, s0, s1 = workloads.materialize(workloads.TensorSpec("split", 0, (n,), 0, 64, 2.0, "normal", seed))
    return s0, s1


def _same(t, e):
    return np.array_equal(t.cpu().numpy(), e)


@pytest.mark.parametrize("tiles", [1, 257, 513, 769, 1024, 1025, 1281, 1537])
@pytest.mark.parametrize("w", [4, 6, 7, 8, 10, 20, 32])
def test_single_tensor(w, tiles):
    k, per = 9, 64 * (64 // w)
    for n in (tiles * per - 1, (tiles - 1) * per + 5):
        s0, s1 = _shares(n, tiles)
        d0, d1 = torch.from_numpy(s0).to(DEV), torch.from_numpy(s1).to(DEV)
        for dealer in (hb.HB_DEALER_PER_GATE, hb.HB_DEALER_SHARED_MASK):
            for call, ref in ((hb.hb_relu_ex, oracle.relu), (hb.hb_drelu_ex, oracle.drelu)):
                r0, r1, bits = call(d0, d1, k, k + w, SEED, dealer)
                e0, e1, ebits = ref(s0, s1, k, k + w, SEED, variant=dealer, threads=8)
                assert _same(r0, e0) and _same(r1, e1) and bits == ebits, (n, dealer, call.__name__)
        r0, r1, _ = hb.hb_sign_shares(d0, d1, k, k + w, SEED)
        e0, e1 = oracle.evaluate(s0, s1, k, k + w, SEED, oracle.WHAT_SIGN, threads=8)
        assert _same(r0, e0) and _same(r1, e1), n


@pytest.mark.parametrize("w", [5, 8])
def test_batch_of_more_tensors_than_a_launch_holds(w):
    k, per = 9, 64 * (64 // w)
    sizes = [900 * per + 5, 7, 200 * per - 1] + [per // 4 * (i % 6) + i for i in range(27)]    # 24 tensors a launch
    host = [_shares(n, i) for i, n in enumerate(sizes)]
    items = []
    for i, (s0, s1) in enumerate(host):
        d0, d1 = torch.from_numpy(s0).to(DEV), torch.from_numpy(s1).to(DEV)
        items.append((d0, d1, torch.empty_like(d0), torch.empty_like(d1), k, k + w, hb.hb_tensor_seed(SEED, i)))
    hb.hb_relu_batch(items)
    for (s0, s1), (_, _, o0, o1, _, _, seed) in zip(host, items):
        e0, e1, _ = oracle.relu(s0, s1, k, k + w, seed, threads=8)
        assert _same(o0, e0) and _same(o1, e1)


@pytest.mark.parametrize("w", [6, 8])
def test_simulator(w):
    k, per = 9, 64 * (64 // w)
    for n in (1024 * per + 5, 1280 * per - 1):
        x = (np.random.default_rng(n).standard_normal(n) * 2).astype(np.float32)
        y = hb.hb_sim_relu_f32(torch.from_numpy(x).to(DEV), k, k + w, SEED, 5)
        assert np.array_equal(y.cpu().numpy(), oracle.sim_relu_f32(x, k, k + w, SEED, 5, threads=8))
