"""The native short cuts of hb.py against the general path that they replace (a call with its stream given goes through ctypes):
same results, same return values, and the same refusals."""
import numpy as np
import pytest
import torch

from paper_2309_04875_amd import hb

pytestmark = pytest.mark.gpu

DEV = "cuda"
N, K, M, SEED = 4099, 12, 20, 0x2309048750000057


def _shares(count=2, n=N):
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    return [torch.randint(-2**62, 2**62, (n,), generator=g, device=DEV, dtype=torch.int64) for _ in range(count)]


def _outs(count=2):
    return [torch.zeros(N, dtype=torch.int64, device=DEV) for _ in range(count)]


def _native_names():
    hb.load()
    return hb._native


class _Counted:
    """Counts the calls that a short cut has served."""

    def __init__(self, monkeypatch, name):
        self.served = 0
        native = getattr(_native_names(), name)

        def call(*args):
            r = native(*args)
            self.served += r is not NotImplemented
            return r
        fake = type("Fake", (), {n: staticmethod(getattr(hb._native, n)) for n in dir(hb._native) if not n.startswith("__")})
        setattr(fake, name, staticmethod(call))
        monkeypatch.setattr(hb, "_native", fake)


def _calls():
    s = _shares(4)
    x = torch.randn(N, device=DEV)
    y = lambda: torch.zeros(N, device=DEV)                                                          # noqa: E731
    ws = lambda d: torch.zeros(hb.hb_party_workspace_bytes_ex(N, K, M, d), dtype=torch.uint8, device=DEV)   # noqa: E731
    items = lambda: [(s[0], s[1], *_outs(), K, M, SEED), (s[2], s[3], *_outs(), 9, 15, SEED + 1)]   # noqa: E731

    def batch(call, *extra):
        def run(**kw):
            b = items()
            return (call(b, *extra, **kw),) + tuple(t for i in b for t in i[2:4])
        return run
    return {
        "relu": ("shares", lambda **kw: hb.hb_relu(s[0], s[1], K, M, SEED, *_outs(), **kw)),
        "drelu": ("shares", lambda **kw: hb.hb_drelu(s[0], s[1], K, M, -3, *_outs(), **kw)),
        "sign": ("shares", lambda **kw: hb.hb_sign_shares(s[0], s[1], 0, 64, 2**70 + 7, *_outs(), **kw)),
        "relu_ex": ("shares", lambda **kw: hb.hb_relu_ex(s[0], s[1], K, M, SEED, 1, *_outs(), **kw)),
        "drelu_ex": ("shares", lambda **kw: hb.hb_drelu_ex(s[0], s[1], K, M, SEED, 0, *_outs(), **kw)),
        "relu_mp": ("parties", lambda **kw: hb.hb_relu_mp(s[:3], K, M, SEED, _outs(3), **kw)),
        "drelu_mp": ("parties", lambda **kw: hb.hb_drelu_mp(s, K, M, SEED, _outs(4), **kw)),
        "batch": ("batch", batch(hb.hb_relu_batch)),
        "drelu_batch_ex": ("batch", batch(hb.hb_drelu_batch_ex, 1)),
        "sim": ("sim_relu", lambda **kw: hb.hb_sim_relu_f32(x, K, M, SEED, 3, y(), **kw)),
        "share": ("share", lambda **kw: hb.hb_share_f32(x, 3, *_outs(), **kw)),
        "reveal": ("reveal", lambda **kw: hb.hb_reveal_f32(s[0], s[1], y(), **kw)),
        "eco": ("eco_scan", lambda **kw: hb.hb_eco_scan(s[0], s[1], torch.zeros(64, dtype=torch.int64, device=DEV), **kw)),
        "party": ("party", lambda **kw: hb.hb_relu_party(s[0], s[1], K, M, SEED, *_outs(), ws(0), **kw)),
        "party_ex": ("party", lambda **kw: hb.hb_relu_party_ex(s[0], s[1], K, M, SEED, 1, *_outs(), ws(1), **kw)),
    }


def _flat(r):
    if isinstance(r, (tuple, list)):
        return [v for e in r for v in _flat(e)]
    return [r]


@pytest.mark.parametrize("name", sorted(("relu", "drelu", "sign", "relu_ex", "drelu_ex", "relu_mp", "drelu_mp", "batch", "drelu_batch_ex",
                                         "sim", "share", "reveal", "eco", "party", "party_ex")))
def test_same_as_general_path(name, monkeypatch):
    cut, call = _calls()[name]
    counted = _Counted(monkeypatch, cut)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                                   # the current stream is asked for at each call
        got = _flat(call())
    assert counted.served == 1
    ref = _flat(call(stream=side))
    assert counted.served == 1
    torch.cuda.synchronize()
    assert len(got) == len(ref)
    for g, r in zip(got, ref):
        assert type(g) is type(r)
        if isinstance(g, torch.Tensor):
            assert g.dtype == r.dtype and g.shape == r.shape and torch.equal(g, r)
        else:
            assert g == r


def test_plan_run(monkeypatch):
    counted = _Counted(monkeypatch, "plan_run")
    s = _shares()
    o, p = _outs(), _outs()
    plan, other = hb.hb_plan_create([(*s, *o, K, M, SEED)]), hb.hb_plan_create([(*s, *p, K, M, SEED)])
    bits = hb.hb_plan_run(plan)
    assert counted.served == 1
    assert bits == hb.hb_plan_run(other, torch.cuda.current_stream()) and counted.served == 1
    assert torch.equal(o[0], p[0]) and torch.equal(o[1], p[1])
    plan.close()
    for st in (None, torch.cuda.current_stream()):
        with pytest.raises(hb.HbError):
            plan.run(st)


@pytest.mark.parametrize("change", ["k_numpy", "k_bool", "out_none", "int32", "strided", "host", "size", "subclass"])
def test_other_forms_are_left_to_the_general_path(change, monkeypatch):
    counted = _Counted(monkeypatch, "shares")
    s, o = _shares(), _outs()
    k = {"k_numpy": np.int64(K), "k_bool": True}.get(change, K)
    error = {"int32": TypeError, "strided": TypeError, "host": TypeError, "size": ValueError}.get(change)
    if change == "out_none":
        o = [None, None]
    elif change == "int32":
        o[0] = o[0].to(torch.int32)
    elif change == "strided":
        o[0] = torch.zeros(2 * N, dtype=torch.int64, device=DEV)[::2]
    elif change == "host":
        s[1] = s[1].cpu()
    elif change == "size":
        o[1] = o[1][:-1]
    elif change == "subclass":
        s[0] = s[0].as_subclass(type("Mine", (torch.Tensor,), {}))
    if error is not None:
        with pytest.raises(error):
            hb.hb_relu(*s, k, M, SEED, *o)
    else:
        r = hb.hb_relu(*s, k, M, SEED, *o)
        e = hb.hb_relu(s[0].as_subclass(torch.Tensor), s[1], int(k), M, SEED, *_outs())
        assert torch.equal(r[0].as_subclass(torch.Tensor), e[0]) and torch.equal(r[1], e[1]) and r[2] == e[2]
        assert counted.served == 1
        return
    assert counted.served == 0


@pytest.mark.parametrize("k,m", [(20, 12), (-1, 8), (0, 65)])
def test_errors_of_the_library(k, m):
    s, o = _shares(), _outs()
    raised = []
    for st in (None, torch.cuda.current_stream()):
        with pytest.raises(hb.HbError) as e:
            hb.hb_relu(*s, k, m, SEED, *o, stream=st)
        raised.append((e.value.status, str(e.value)))
    assert raised[0] == raised[1]
    with pytest.raises(hb.HbError):
        hb.hb_relu(*s, K, M, SEED, o[0], o[0])                     # outputs overlap


# A call with every argument given, as (short cut, function, arguments); a list of tensors is an argument of one call among parties.
def _full_calls():
    s, x, y = _shares(4), torch.randn(N, device=DEV), torch.zeros(N, device=DEV)
    workspace = [torch.zeros(hb.hb_party_workspace_bytes_ex(N, K, M, d), dtype=torch.uint8, device=DEV) for d in (0, 1)]
    counts = torch.zeros(64, dtype=torch.int64, device=DEV)
    return {
        "relu": ("shares", hb.hb_relu, [s[0], s[1], K, M, SEED, *_outs()]),
        "drelu": ("shares", hb.hb_drelu, [s[0], s[1], K, M, SEED, *_outs()]),
        "sign": ("shares", hb.hb_sign_shares, [s[0], s[1], K, M, SEED, *_outs()]),
        "relu_ex": ("shares", hb.hb_relu_ex, [s[0], s[1], K, M, SEED, 1, *_outs()]),
        "drelu_ex": ("shares", hb.hb_drelu_ex, [s[0], s[1], K, M, SEED, 1, *_outs()]),
        "relu_mp": ("parties", lambda a, b, c, *rest, **kw: hb.hb_relu_mp([a, b, c], *rest[:3], list(rest[3:]), **kw), [*s[:3], K, M, SEED, *_outs(3)]),
        "drelu_mp": ("parties", lambda a, b, c, *rest, **kw: hb.hb_drelu_mp([a, b, c], *rest[:3], list(rest[3:]), **kw), [*s[:3], K, M, SEED, *_outs(3)]),
        "batch": ("batch", lambda a, b, k, m, seed, c, d, **kw: hb.hb_relu_batch([(a, b, c, d, k, m, seed)], **kw), [s[0], s[1], K, M, SEED, *_outs()]),
        "drelu_batch_ex": ("batch", lambda a, b, k, m, seed, c, d, **kw: hb.hb_drelu_batch_ex([(a, b, c, d, k, m, seed)], 1, **kw), [s[0], s[1], K, M, SEED, *_outs()]),
        "sim": ("sim_relu", hb.hb_sim_relu_f32, [x, K, M, SEED, 3, y]),
        "share": ("share", hb.hb_share_f32, [x, 3, *_outs()]),
        "reveal": ("reveal", hb.hb_reveal_f32, [s[0], s[1], y]),
        "eco": ("eco_scan", hb.hb_eco_scan, [s[0], s[1], counts]),
        "party": ("party", hb.hb_relu_party, [s[0], s[1], K, M, SEED, *_outs(), workspace[0]]),
        "party_ex": ("party", hb.hb_relu_party_ex, [s[0], s[1], K, M, SEED, 1, *_outs(), workspace[1]]),
    }


CHANGES = {
    "type": lambda t: t.to(torch.float64 if t.dtype == torch.float32 else torch.int8 if t.dtype == torch.uint8 else torch.int32),
    "host": lambda t: t.cpu(),
    "strided": lambda t: t.repeat_interleave(2)[::2],
    "short": lambda t: t[:-1],
}


@pytest.mark.parametrize("change", sorted(CHANGES))
@pytest.mark.parametrize("name", sorted(("relu", "drelu", "sign", "relu_ex", "drelu_ex", "relu_mp", "drelu_mp", "batch", "drelu_batch_ex",
                                         "sim", "share", "reveal", "eco", "party", "party_ex")))
def test_every_tensor_of_every_call_is_checked(name, change, monkeypatch):
    cut, call, args = _full_calls()[name]
    counted = _Counted(monkeypatch, cut)
    call(*args)
    assert counted.served == 1
    for i, arg in enumerate(args):
        if not isinstance(arg, torch.Tensor):
            continue
        given = args[:i] + [CHANGES[change](arg)] + args[i + 1:]
        raised = []
        for kw in ({}, {"stream": torch.cuda.current_stream()}):
            with pytest.raises((TypeError, ValueError, hb.HbError)) as e:
                call(*given, **kw)
            raised.append((type(e.value), str(e.value)))
        assert raised[0] == raised[1] and counted.served == 1, (i, raised)


def test_forms_of_sets_and_parties(monkeypatch):
    counted = _Counted(monkeypatch, "batch")
    s = _shares(4)
    assert hb.hb_relu_batch([]) == hb.hb_relu_batch([], torch.cuda.current_stream()) == 0
    served = counted.served
    item = (*s[:2], *_outs(), K, M, SEED)
    assert hb.hb_relu_batch([list(item)]) == hb.hb_relu_batch([item], torch.cuda.current_stream())    # a list for a tuple: as before
    for wrong in ([item[:6]], [item + (1,)]):
        with pytest.raises(ValueError):
            hb.hb_relu_batch(wrong)
    with pytest.raises(TypeError):
        hb.hb_relu_batch_ex([item], None)
    assert counted.served == served
    for count in (1, 5, 9):                                        # 9: more than the short cut takes
        raised = []
        for kw in ({}, {"stream": torch.cuda.current_stream()}):
            with pytest.raises(hb.HbError) as e:
                hb.hb_relu_mp(_shares(count), K, M, SEED, _outs(count), **kw)
            raised.append(str(e.value))
        assert raised[0] == raised[1]
    with pytest.raises(ValueError):
        hb.hb_relu_mp(s[:3], K, M, SEED, _outs(2))


def test_nothing_is_enqueued_before_a_call_is_left_to_the_general_path():
    from torch.utils._python_dispatch import TorchDispatchMode
    s, o = _shares(), _outs()
    workspace = torch.zeros(hb.hb_party_workspace_bytes(N, K, M), dtype=torch.uint8, device=DEV)
    hb.load()
    hb.hb_relu_party(*s, K, M, SEED, *_outs(), workspace)            # the native code is loaded by the first call of all

    class Refuses(TorchDispatchMode):
        written = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            if "view" in str(func):
                self.written.append(bool(torch.count_nonzero(o[0])))
                raise RuntimeError("no views")
            return func(*args, **(kwargs or {}))
    with pytest.raises(RuntimeError, match="no views"):
        with Refuses():
            hb.hb_relu_party(*s, K, M, SEED, *o, workspace)
    assert Refuses.written == [False, True]                         # the short cut's try, then the general path's, after its launch
