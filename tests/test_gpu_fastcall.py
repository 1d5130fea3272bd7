"""The native half of the binding against its ctypes half, on device tensors: both are bound to functions that note their arguments and
launch nothing, so that a check that is missing shows as a call that should not have been made."""
import ctypes
import inspect
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2407_18121_amd import binding as ec

pytestmark = pytest.mark.gpu
B, H, T, D, P, N, CAP, L = 2, 4, 6, 64, 3, 5, 9, 7


class Sub(torch.Tensor):
    pass


def _calls(dt, G):
    """Arguments of a usual call of every entry point that the native half has."""
    t = lambda *s, dtype=dt: torch.zeros(s, dtype=dtype, device="cuda")
    f, i = (lambda *s: t(*s, dtype=torch.float32)), (lambda *s: t(*s, dtype=torch.int32))
    prompt = lambda: dict(q=t(B, H, T, D), k=t(B, H, T, D), v=t(B, H, T, D), out=t(B, H, T, D), lse=f(B, H, T), score=f(B, G, T))
    step = lambda: dict(q=t(B, H, D), k_new=t(B, H, D), v_new=t(B, H, D), k_cache=t(B, H, CAP, D), v_cache=t(B, H, CAP, D), pos=i(B, G, CAP))
    return {
        "prefill_score": dict(prompt(), scale=0.3, ws=f(40)),
        "prefill_score_varlen": dict(prompt(), seq_len=i(B), scale=0.3, ws=f(40)),
        "chunk_score": dict(prompt(), k=t(B, H, P + T + 2, D), v=t(B, H, P + T + 2, D), score=f(B, G, P + T), P=P, scale=0.3, ws=f(40)),
        "select_anchors": dict(score=f(B, G, T), n_anchor=N, protect_first=1, protect_last=2, anchor_idx=i(B, G, N)),
        "merge_compact": dict(k=t(B, H, T, D), v=t(B, H, T, D), anchor_idx=i(B, G, N), k_cache=t(B, H, CAP, D), v_cache=t(B, H, CAP, D),
                              counts=i(B, G, N), assign=i(B, G, T), pos=i(B, G, CAP), merge_mode=1),
        "remerge_compact": dict(k=t(B, H, T + 4, D), v=t(B, H, T + 4, D), L=L, anchor_idx=i(B, G, N), k_cache=t(B, H, CAP, D), v_cache=t(B, H, CAP, D),
                                weights=i(B, G, L), src_pos=i(B, G, L), counts=i(B, G, N), assign=i(B, G, L), pos=i(B, G, CAP), merge_mode=1),
        "decode_step": dict(step(), cache_len=7, evict_idx=2, new_pos=11, scale=0.3, out=t(B, H, D), ws=f(40), G=G),
        "decode_step_varlen": dict(step(), cache_len_b=i(B), evict_idx_b=i(B), new_pos_b=i(B), scale=0.3, out=t(B, H, D), G=G, ws=f(40)),
        "decode_score_step": dict(step(), freq=f(B, G, CAP), cache_len=7, new_pos=11, scale=0.3, out=t(B, H, D), ws=f(40)),
        "evict_min": dict(k_cache=t(B, H, CAP, D), v_cache=t(B, H, CAP, D), pos=i(B, G, CAP), freq=f(B, G, CAP), length=8, protect_first=1,
                          protect_recent=2, victim=i(B, G)),
    }


@pytest.fixture
def noted(monkeypatch):
    """(native, ctypes): functions that make a call through one half and return what the library would have been given, or None where the
    native half left it, or the error of the ctypes half."""
    lib, fast, seen, stubs = ec.load(), ec._fast, [], {}
    assert fast is not None
    for name in ec._FAST:
        fn = getattr(lib, "ec_" + name)
        stubs["ec_" + name] = ctypes.CFUNCTYPE(ctypes.c_int, *fn.argtypes)(lambda *a, name=name: seen.append((name, *a)) or 0)
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value

    def native(name, args):
        order = [p for p in inspect.signature(getattr(ec, "ec_" + name)).parameters if p != "check"]
        rc = getattr(fast, name)(*(args[p] for p in order))
        assert rc == (0 if seen else None)
        return seen.pop() if seen else None

    def through_ctypes(name, args):
        try:
            getattr(ec, "ec_" + name)(**args)
        except Exception as e:
            assert not seen
            return e
        return seen.pop()
    fast.bind(ec._raw_stream, ec._device, tuple(address(stubs["ec_" + n]) for n in ec._FAST))
    monkeypatch.setattr(ec, "_fast", None)
    monkeypatch.setattr(ec, "load", lambda: SimpleNamespace(**stubs))
    yield native, through_ctypes
    fast.bind(ec._raw_stream, ec._device, tuple(address(getattr(lib, "ec_" + n)) for n in ec._FAST))


@pytest.mark.parametrize("name", ec._FAST)
@pytest.mark.parametrize("dt,G", [(torch.bfloat16, 1), (torch.float32, H)])
def test_usual_calls(noted, name, dt, G):
    """Both halves hand the library the same; none of these calls is left to ctypes."""
    native, through_ctypes = noted
    good = _calls(dt, G)[name]
    optional = [p for p in ("out", "lse", "counts", "assign", "pos", "weights", "src_pos", "evict_idx_b", "new_pos_b", "ws", "G")
                if p in good and not (p == "out" and name.startswith("decode"))]
    usual = [good] + [dict(good, **{p: None}) for p in optional]
    if "scale" in good:  # what a program computes a scale with
        usual += [dict(good, scale=s) for s in (1.0 / np.sqrt(D), np.float64(0.125), 1, 1e30)]
    usual += [dict(good, **{p: True}) for p, x in good.items() if type(x) is int and p not in ("P", "n_anchor", "L", "G")]
    for args in usual:
        got = native(name, args)
        assert got is not None and got == through_ctypes(name, args)


def _others(x):
    """Values that may be wrong in the place of x."""
    yield None
    yield "text"
    if isinstance(x, torch.Tensor):
        yield 3
        for d in range(x.dim()):
            yield x.new_zeros([n + (i == d) for i, n in enumerate(x.shape)])
        yield x.new_zeros((*x.shape, 1))
        yield x.new_zeros((*x.shape, 2))[..., 0]           # not contiguous
        yield x.cpu()
        yield x.to("meta")
        yield x.as_subclass(Sub)
        yield x.expand(2, *x.shape)[0] if x.dim() else x   # usual
        yield from (x.to(t) for t in (torch.float32, torch.bfloat16, torch.float16, torch.int32, torch.int64, torch.uint8))
    else:
        yield from (3.0, -7, 0, 1, 2, 1 << 31, 1 << 40, -(1 << 70), np.int64(3), np.float32(0.5), torch.ones(1), float("nan"))


@pytest.mark.parametrize("name", ec._FAST)
@pytest.mark.parametrize("dt,G", [(torch.bfloat16, 1), (torch.float32, H)])
def test_every_argument_replaced(noted, name, dt, G):
    """Whatever the ctypes half words an error about, the native half leaves to it; what it takes itself reaches the library alike."""
    native, through_ctypes = noted
    good = _calls(dt, G)[name]
    for p, x in good.items():
        refused = 0
        for other in _others(x):
            args = dict(good, **{p: other})
            got, want = native(name, args), through_ctypes(name, args)
            if isinstance(want, Exception):
                assert got is None, (p, other)
                refused += 1
            elif got is not None:
                assert repr(got) == repr(want), (p, other)  # a scale may be NaN
        # a workspace may be of any type and shape: the library checks its size
        assert refused >= (3 if p == "ws" else 8 if isinstance(x, torch.Tensor) else 1), (p, refused)
