"""The work whose speed matters: what users of the library have it do, one case per kind of use.

A case names the call (`kind`), the sizes, the slice [k, m) and the options; `prepare` makes the device buffers that a
program holds before the call, `run` is one pass through the public entry points, `work` is what that pass cannot do
without.  Sizes are the five named workloads of bench.py (flat 65,536; ResNet18 on 3x32x32 images, one image and batch
512; the 2^26 width sweep; ResNet18 on 3x224x224 images, batch 64) and generic ones beside them.  Inputs are the
seeded activations of paper_2309_04875_amd.workloads: Gaussian or Laplace values at 2^16 fixed point, share0 uniform.

Everything is integer arithmetic on Z_2^64 (the simulator's floats are decoded from it), so results are exact.
"""
import math

import torch

from paper_2309_04875_amd import hb, workloads

DEV = "cuda"
PER_GATE, SHARED = hb.HB_DEALER_PER_GATE, hb.HB_DEALER_SHARED_MASK


def listed():
    return [
        # One small layer through the plain call: arguments are checked on every call, so host time and launch latency count.
        {"name": "relu_flat_64k", "kind": "flat", "op": "relu", "n": 65536, "k": 12, "m": 20, "dealer": PER_GATE, "dist": "normal", "offset": 0},
        # Latency of a whole network: the 17 ReLU layers of one 32x32 image, prepared once and issued every step.
        {"name": "plan_cifar_one_image", "kind": "plan", "net": "cifar", "batch": 1, "k": -1, "m": -1, "search": 2, "dealer": PER_GATE},
        # Throughput: the same 17 layers at batch 512 in one batched call (bench.py's headline).
        {"name": "batch_cifar_512", "kind": "set", "net": "cifar", "batch": 512, "k": 12, "m": 20, "search": 3, "dealer": PER_GATE},
        # Layers with different slice widths (6, 8, 10): ResNet18 on 224x224 images, batch 64, searched (k, m) per layer.
        {"name": "batch_imagenet_64_mixed_widths", "kind": "set", "net": "imagenet", "batch": 64, "k": -1, "m": -1, "search": 5, "dealer": PER_GATE},
        # No slicing: the exact ReLU on the full ring, the baseline every reduced ring is compared with.
        {"name": "relu_full_ring_2e26", "kind": "flat", "op": "relu", "n": 1 << 26, "k": 0, "m": 64, "dealer": PER_GATE, "dist": "laplace", "offset": 0},
        # A middle width on the dealer layout that opens 3w bits a round, odd size, as a slice of a larger buffer.
        {"name": "relu_w16_shared_mask_odd", "kind": "flat", "op": "relu", "n": 9999991, "k": 8, "m": 24, "dealer": SHARED, "dist": "laplace", "offset": 1},
        # The comparison alone (max-pooling, arg-max and masks are built on it), a narrow slice, odd size.
        {"name": "drelu_w6_odd", "kind": "flat", "op": "drelu", "n": 3211267, "k": 10, "m": 16, "dealer": PER_GATE, "dist": "normal", "offset": 0},
        # The messages of a two-GPU run: every opening through packed wires in memory, a mid-size layer.
        {"name": "party_layer_w8", "kind": "party", "n": 64 * 128 * 16 * 16, "k": 12, "m": 20, "dealer": PER_GATE},
        # Three parties, an odd size.
        {"name": "relu_three_parties_odd", "kind": "mp", "op": "relu", "parties": 3, "n": 4194304 + 1003, "k": 12, "m": 20},
        # The single-node simulator's layer: plaintext floats through the protocol, batch 64 of the first 32x32 layer.
        {"name": "sim_relu_f32", "kind": "sim", "n": 64 * 64 * 32 * 32, "k": 12, "m": 20},
        # The zero-error search: mismatches of every high cut over one layer of a validation batch.
        {"name": "eco_scan_layer", "kind": "eco", "n": 16 * 64 * 112 * 112},
        # Float boundary around the protocol: share a layer's floats, ReLU on the shares, reveal floats; one 224x224 image's first layer.
        {"name": "share_relu_reveal_one_image", "kind": "boundary", "n": 64 * 112 * 112, "k": 9, "m": 19},
    ]


def _size(rng, lo, hi):
    """Log-uniform in [lo, hi]; half of the sizes as they fall (odd ones among them), the others rounded to a multiple of 64."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        n = max(64, n // 64 * 64)
    return n


def _slice(rng):
    """A slice as layers are given them: mostly widths 4 to 10, sometimes a middle one or the full ring."""
    w = rng.choice([4, 5, 6, 6, 7, 8, 8, 8, 9, 10, 10, 12, 16, 20, 24, 32, 48, 64])
    k = rng.randint(6, 16) if w <= 32 else rng.randint(0, 64 - w)
    return k, k + w


def draw(rng):
    kind = rng.choice(["flat", "flat", "flat", "plan", "set", "set", "party", "mp", "sim", "eco", "boundary"])
    k, m = _slice(rng)
    dealer = rng.choice([PER_GATE, PER_GATE, SHARED])
    if kind == "flat":
        op = rng.choice(["relu", "relu", "drelu", "sign"])
        return {"kind": kind, "op": op, "n": _size(rng, 1 << 13, 1 << 26), "k": k, "m": m, "dealer": PER_GATE if op == "sign" else dealer,
                "dist": rng.choice(["normal", "laplace"]), "offset": rng.choice([0, 0, 1])}
    if kind in ("plan", "set"):
        net = rng.choice(["cifar", "imagenet"])
        top = (8 if net == "cifar" else 2) if kind == "plan" else (512 if net == "cifar" else 64)
        batch = min(top, int(math.exp(rng.uniform(0.0, math.log(top + 1)))))
        fixed = rng.random() < 0.5 and m - k <= 32
        return {"kind": kind, "net": net, "batch": batch, "k": k if fixed else -1, "m": m if fixed else -1, "search": rng.randint(1, 999), "dealer": dealer}
    if kind == "party":
        return {"kind": kind, "n": _size(rng, 1 << 12, 1 << 23), "k": k, "m": m, "dealer": dealer}
    if kind == "mp":
        return {"kind": kind, "op": rng.choice(["relu", "relu", "drelu"]), "parties": rng.choice([3, 4]),
                "n": _size(rng, 1 << 14, 1 << 24 if m - k <= 10 else 1 << 22), "k": k, "m": m}
    if kind == "sim":
        return {"kind": kind, "n": _size(rng, 1 << 14, 1 << 25), "k": k, "m": m}
    if kind == "eco":
        return {"kind": kind, "n": _size(rng, 1 << 14, 1 << 26)}
    return {"kind": kind, "n": _size(rng, 1 << 14, 1 << 24), "k": k, "m": m}


# ---- what a program holds before the call ------------------------------------------------------------------------

def _specs(case, seed):
    """The 17 layers of a set case; k < 0: every layer its own (k, m), those that the workload draws for `search`."""
    make = workloads.resnet18_cifar if case["net"] == "cifar" else workloads.resnet18_imagenet
    own = case["k"] < 0
    return [workloads.TensorSpec(s.workload, s.tensor_id, s.shape, s.k if own else case["k"], s.m if own else case["m"],
                                 s.sigma, s.dist, 100 * seed + s.tensor_id)
            for s in make(case["batch"], case["search"])]


def _flat(case, seed, sigma=2.0):
    """Shares of a flat tensor and output buffers; offset 1 places all four at an odd element of larger buffers."""
    off = case.get("offset", 0)
    dist = case.get("dist", "normal")
    spec = workloads.TensorSpec("flat", 0, (case["n"] + off,), 0, 64, sigma if dist == "normal" else 1.0, dist, 7 + seed)
    _, s0, s1 = workloads.materialize_on_device(spec, DEV)
    o0, o1 = torch.empty_like(s0), torch.empty_like(s1)
    return s0[off:], s1[off:], o0[off:], o1[off:]


def _dealer_seed(seed):
    return hb.hb_tensor_seed(0x2309048750000001, seed)


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case, "seed": _dealer_seed(seed)}
    if kind == "flat":
        state["shares"] = _flat(case, seed)
    elif kind in ("plan", "set"):
        layers = []
        for spec in _specs(case, seed):
            _, s0, s1 = workloads.materialize_on_device(spec, DEV)
            layers.append((s0, s1, torch.empty_like(s0), torch.empty_like(s1), spec.k, spec.m, hb.hb_tensor_seed(state["seed"], spec.tensor_id)))
        state["layers"] = layers
        if kind == "plan":
            state["plan"] = hb.hb_plan_create(layers, True, case["dealer"])
    elif kind == "party":
        state["shares"] = _flat(case, seed)
        state["workspace"] = torch.empty(hb.hb_party_workspace_bytes_ex(case["n"], case["k"], case["m"], case["dealer"]), dtype=torch.uint8, device=DEV)
    elif kind == "mp":
        s0, s1, o0, o1 = _flat(case, seed)
        g = torch.Generator(device=DEV)
        g.manual_seed(99 + seed)
        shares = [s0, s1]
        for _ in range(case["parties"] - 2):      # split share1 once more: the sum over the parties stays x
            r = (torch.randint(0, 1 << 32, (case["n"],), generator=g, device=DEV, dtype=torch.int64) << 32) | \
                torch.randint(0, 1 << 32, (case["n"],), generator=g, device=DEV, dtype=torch.int64)
            shares[1] = shares[1] - r
            shares.append(r)
        state["shares"], state["outs"] = shares, [torch.empty_like(s) for s in shares]
    elif kind in ("sim", "boundary"):
        g = torch.Generator(device=DEV)
        g.manual_seed(11 + seed)
        state["x"] = torch.randn(case["n"], generator=g, device=DEV, dtype=torch.float32) * 2.0
        state["y"] = torch.empty_like(state["x"])
        state["share_seed"] = hb.hb_tensor_seed(state["seed"], 1)
        if kind == "boundary":
            state["shares"] = tuple(torch.empty(case["n"], dtype=torch.int64, device=DEV) for _ in range(4))
    elif kind == "eco":
        state["shares"] = _flat(case, seed)[:2]
        state["counts"] = torch.empty(64, dtype=torch.int64, device=DEV)
    else:
        raise ValueError(kind)
    return state


# ---- one pass ----------------------------------------------------------------------------------------------------

def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "flat":
        s0, s1, o0, o1 = state["shares"]
        if case["op"] == "sign":
            hb.hb_sign_shares(s0, s1, case["k"], case["m"], state["seed"], o0, o1)
        elif case["dealer"] != PER_GATE:
            call = hb.hb_relu_ex if case["op"] == "relu" else hb.hb_drelu_ex
            call(s0, s1, case["k"], case["m"], state["seed"], case["dealer"], o0, o1)
        else:
            call = hb.hb_relu if case["op"] == "relu" else hb.hb_drelu
            call(s0, s1, case["k"], case["m"], state["seed"], o0, o1)
        return o0, o1
    if kind == "plan":
        hb.hb_plan_run(state["plan"])
        return [t for layer in state["layers"] for t in layer[2:4]]
    if kind == "set":
        if case["dealer"] != PER_GATE:
            hb.hb_relu_batch_ex(state["layers"], case["dealer"])
        else:
            hb.hb_relu_batch(state["layers"])
        return [t for layer in state["layers"] for t in layer[2:4]]
    if kind == "party":
        s0, s1, o0, o1 = state["shares"]
        if case["dealer"] != PER_GATE:
            return hb.hb_relu_party_ex(s0, s1, case["k"], case["m"], state["seed"], case["dealer"], o0, o1, state["workspace"])
        return hb.hb_relu_party(s0, s1, case["k"], case["m"], state["seed"], o0, o1, state["workspace"])
    if kind == "mp":
        call = hb.hb_relu_mp if case["op"] == "relu" else hb.hb_drelu_mp
        return call(state["shares"], case["k"], case["m"], state["seed"], state["outs"])
    if kind == "sim":
        return hb.hb_sim_relu_f32(state["x"], case["k"], case["m"], state["seed"], state["share_seed"], state["y"])
    if kind == "eco":
        return hb.hb_eco_scan(state["shares"][0], state["shares"][1], state["counts"])
    s0, s1, r0, r1 = state["shares"]
    hb.hb_share_f32(state["x"], state["share_seed"], s0, s1)
    hb.hb_relu(s0, s1, case["k"], case["m"], state["seed"], r0, r1)
    return hb.hb_reveal_f32(r0, r1, state["y"]), r0, r1


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def _ops(op, w, dealer=PER_GATE, parties=2):
    """64-bit integer operations per element: a dealer word is one SplitMix64 output (add, three shifts, three xors, two
    multiplies), a Beaver AND about nine bitwise operations per party, the result of an element about ten operations per
    party plus the products of its multiply."""
    if parties == 2:
        lanes = min(64 // w, 32)
    else:
        lanes = min(64 // w, 64 // parties)
    rounds = 0 if w == 1 else (w - 1).bit_length()
    gates = 2 * rounds if rounds else 1                  # the last round's propagate gate feeds nothing
    gate_words = 3 * parties - 1
    circuit = (parties - 1) * gates * (gate_words * 9 + 9 * parties)
    if dealer == SHARED:
        circuit -= max(rounds - 1, 0) * 2 * 9            # one mask (two words) for both gates of a round
    words = 0 if op == "sign" else (parties - 1 if op == "drelu" else 4 * parties - 2)
    finish = 0 if op == "sign" else 5 * parties + (0 if op == "drelu" else 9 * parties + 3)
    return (circuit + 9) / lanes + 9 * words + finish


def work(case):
    kind = case["kind"]
    if kind in ("plan", "set"):
        specs = _specs(case, 0)
        return {"bytes": 32 * sum(s.n for s in specs), "flops": sum(s.n * _ops("relu", s.w, case["dealer"]) for s in specs)}
    n = case["n"]
    if kind == "eco":
        return {"bytes": 16 * n + 512, "flops": 3 * n + 4 * n}          # sum, sign word, a carry-save step of the counters
    w = case["m"] - case["k"]
    if kind == "flat":
        return {"bytes": 32 * n, "flops": n * _ops(case["op"], w, case["dealer"])}
    if kind == "party":
        # shares in, result shares and both wires out
        return {"bytes": 32 * n + 16 * hb.hb_party_wire_words_ex(n, case["k"], case["m"], case["dealer"]),
                "flops": n * _ops("relu", w, case["dealer"])}
    if kind == "mp":
        return {"bytes": 16 * case["parties"] * n, "flops": n * _ops(case["op"], w, PER_GATE, case["parties"])}
    if kind == "sim":
        return {"bytes": 8 * n, "flops": n * (_ops("relu", w) + 14)}     # plus one word, encode and decode
    # boundary: 4 + 16 bytes to share, 32 for the ReLU, 16 + 4 to reveal
    return {"bytes": 72 * n, "flops": n * (_ops("relu", w) + 14)}


def tolerance(case):
    """Shares, wires and counts are integers, and the simulator's floats are decoded from them."""
    return "exact"
