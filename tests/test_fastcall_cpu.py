"""The binding's native half without a device: tensors on the host make it answer None whatever else is right or wrong with a call
(each argument by itself, on device tensors: test_gpu_fastcall.py), and so does a wrong number of arguments; the binding without it."""
import sys

import pytest
import torch

import paper_2407_18121_amd
from paper_2407_18121_amd import binding as ec


class Sub(torch.Tensor):
    pass


def _steps():
    B, H, cap, D = 2, 4, 12, 64
    x, kc = torch.zeros((B, H, D)), torch.zeros((B, H, cap, D))
    good = dict(q=x, k_new=x, v_new=x, k_cache=kc, v_cache=kc, pos=None, cache_len=3, evict_idx=-1, new_pos=0, scale=0.1, out=x, ws=None, G=1)
    yield good  # on the host
    for name, value in (("q", None), ("q", 3), ("q", x.as_subclass(Sub)), ("k_cache", x), ("v_new", x.bfloat16()), ("out", x.to("meta")),
                        ("k_cache", kc.transpose(2, 3)), ("cache_len", 3.0), ("cache_len", 1 << 40), ("scale", 1), ("G", 3), ("pos", x)):
        yield dict(good, **{name: value})


@pytest.mark.parametrize("i", range(13))
def test_unusual_calls_are_left_to_python(i):
    """Nothing but None, and no exception, for whatever comes in the place of an argument."""
    ec.load()
    assert ec._fast.decode_step(*list(_steps())[i].values()) is None


def test_number_of_arguments():
    ec.load()
    for name in ec._FAST:
        assert getattr(ec._fast, name)() is None


@pytest.mark.parametrize("why", ["missing", "another torch"])
def test_library_without_a_native_half(monkeypatch, why):
    """The library alone is enough: every call goes through ctypes then."""
    ec.load()
    if why == "missing":  # importing it fails
        monkeypatch.setitem(sys.modules, "paper_2407_18121_amd._fastcall", None)
        monkeypatch.delattr(paper_2407_18121_amd, "_fastcall")
    else:
        monkeypatch.setattr(sys.modules["paper_2407_18121_amd._fastcall"], "built_for", "1.0")
    monkeypatch.setattr(ec, "_lib", None)
    monkeypatch.setattr(ec, "_fast", ec._fast)
    with pytest.warns(RuntimeWarning, match="native half"):
        lib = ec.load()
    assert ec._fast is None and lib.ec_evict_index(10, 6, 1, 2, 0, 0, 0, 25, 0, 1) == ec.ec_evict_index(10, 6, 1, 2)
    with pytest.raises(ValueError, match="device memory"):  # through ctypes, up to the device check
        ec.ec_select_anchors(torch.zeros(1, 1, 8), 2, 1, 1, torch.zeros(1, 1, 2, dtype=torch.int32), check=False)
