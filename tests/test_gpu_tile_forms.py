"""Every width from 1 to 32 in every form of a tile launch, all operations, bit for bit against the oracle: whole tiles only
(HB_SMALL_TILE_LIMIT=0), quarters only (a limit above every size), and the rule's own choice where a launch is mixed (three
tiles after a full round of 1024; 700, where a third round of quarters is shared out) or whole (900 after one, more than any width
shares out, so that every width's whole tiles run with dealer words in step where they have that form).  The variable is read
once, so each runs in a child process."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import os, sys
import numpy as np, torch, oracle
from paper_2309_04875_amd import hb
part, rule = sys.argv[1:3]
rng = np.random.default_rng(77)
dev = "cuda"
SEED = 0x2309048750000099
THREADS = 8

def same(what, got, ref):
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r), what

for w in range(1, 33):
    for parties in ((2,) if part == "two" else (3, 4)):
        L = min(64 // w, 32) if parties == 2 else min(64 // w, 64 // parties)
        per = (64 if w >= 4 else 32) * L
        sizes = (1, L + 1, 16 * L + 1, per - 1, per, 5 * per + 17) if rule == "given" else (1027 * per + 5, 1724 * per + 5, 1924 * per - 5)
        for n in sizes:
            k = int(rng.integers(0, 64 - w + 1)); m = k + w
            off = n % 2                                        # odd sizes on buffers that are only 8-byte aligned
            host = [rng.integers(0, 1 << 64, n + off, dtype=np.uint64).view(np.int64) for _ in range(parties)]
            d = [torch.from_numpy(h).to(dev)[off:] for h in host]
            s = [h[off:] for h in host]
            if parties > 2:
                outs, _ = hb.hb_relu_mp(d, k, m, SEED)
                same(("mp relu", parties, w, n), outs, oracle.mp_evaluate(s, k, m, SEED, oracle.WHAT_RELU, threads=THREADS))
                outs, _ = hb.hb_drelu_mp(d, k, m, SEED)
                same(("mp drelu", parties, w, n), outs, oracle.mp_evaluate(s, k, m, SEED, oracle.WHAT_DRELU, threads=THREADS))
                continue
            for layout in (hb.HB_DEALER_PER_GATE, hb.HB_DEALER_SHARED_MASK):
                for call, ref in ((hb.hb_relu_ex, oracle.relu), (hb.hb_drelu_ex, oracle.drelu)):
                    same((call.__name__, layout, w, n), call(d[0], d[1], k, m, SEED, layout)[:2],
                         ref(s[0], s[1], k, m, SEED, variant=layout, threads=THREADS)[:2])
                o = [torch.empty_like(t) for t in d]
                hb.hb_relu_batch_ex([(d[0], d[1], o[0], o[1], k, m, SEED)], layout)
                same(("batch", layout, w, n), o, oracle.relu(s[0], s[1], k, m, SEED, variant=layout, threads=THREADS)[:2])
            same(("sign", w, n), hb.hb_sign_shares(d[0], d[1], k, m, SEED)[:2],
                 oracle.evaluate(s[0], s[1], k, m, SEED, oracle.WHAT_SIGN, threads=THREADS))
            x = (rng.standard_normal(n) * 2).astype(np.float32)
            y = hb.hb_sim_relu_f32(torch.from_numpy(x).to(dev), k, m, SEED, 5)
            assert np.array_equal(y.cpu().numpy(), oracle.sim_relu_f32(x, k, m, SEED, 5, threads=THREADS)), ("sim", w, n)
    print("w", w, flush=True)
print("tile forms ok")
"""


@pytest.mark.parametrize("part", ["two", "more"])
@pytest.mark.parametrize("limit", ["0", "1000000000", None])
def test_every_width_in_every_form(part, limit):
    env = dict(os.environ, PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    env.pop("HB_SMALL_TILE_LIMIT", None)
    if limit is not None:
        env["HB_SMALL_TILE_LIMIT"] = limit
    proc = subprocess.run([sys.executable, "-c", CHILD, part, "own" if limit is None else "given"], env=env, cwd=ROOT,
                          stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert proc.returncode == 0 and "tile forms ok" in proc.stdout, proc.stdout[-2000:]
