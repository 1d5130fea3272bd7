"""Scoring calls whose tensors do not start on a 16-byte boundary: every geometry, element type and head size, any of the
tensors alone and all of them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_18121_amd import binding as ec
from paper_2407_18121_amd import synthetic as syn
from util import assert_close, to_dev, to_host, torch_dtype

pytestmark = pytest.mark.gpu


def _shifted(x, elements):
    """The same tensor `elements` elements into its storage, NaN before and behind it."""
    room = torch.full((x.numel() + 16,), float("nan"), dtype=x.dtype, device="cuda")
    t = room[elements:elements + x.numel()].view(x.shape)
    t.copy_(x)
    return t


@pytest.mark.parametrize("off", [(1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 3, 0), (0, 0, 0, 1), (1, 2, 5, 7)])
@pytest.mark.parametrize("B,H,Tq,P,lens", [
    (1, 2, 200, 0, None), (1, 3, 641, 0, None), (2, 2, 1, 300, None), (1, 2, 130, 77, None), (3, 2, 257, 0, [257, 0, 64]),
    (4, 32, 385, 0, None),  # the aligned launch takes tiles in pairs
])
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_score_of_rows_off_the_16_byte_grid(dtype, D, B, H, Tq, P, lens, off):
    L = P + Tq
    cfg = syn.custom("t", H=H, D=D, B=B, T=L, dtype=dtype, cid=4900 + L)
    q, k, v = syn.prompt_qkv(cfg)
    q = np.ascontiguousarray(q[:, :, P:])
    dq, dk, dv = (_shifted(to_dev(x, dtype), n) for x, n in zip((q, k, v), off))
    out = _shifted(torch.full((B, H, Tq, D), 5.0, dtype=torch_dtype(dtype), device="cuda"), off[3])
    lse = torch.zeros((B, H, Tq), device="cuda") if off[0] else None
    score = torch.zeros((B, H, L), device="cuda")
    ws = ec.new_workspace(ec.EC_FN_PREFILL_SCORE, B, H, L, D, ec.dtype_code(dq))
    if lens:
        ec.ec_prefill_score_varlen(dq, dk, dv, out, lse, score, torch.tensor(lens, dtype=torch.int32, device="cuda"), cfg.scale, ws)
    else:
        ec.ec_chunk_score(dq, dk, dv, P, out, lse, score, cfg.scale, ws)
    torch.cuda.synchronize()
    for b, n in enumerate(lens or [Tq] * B):
        if n:
            ref = oracle.chunk_score(q[b:b + 1, :, :n], k[b:b + 1, :, :P + n], v[b:b + 1, :, :P + n], P, cfg.scale, H)
            assert_close(to_host(out[b:b + 1, :, :n]), ref["out"], dtype, "out")
            assert_close(to_host(score[b:b + 1, :, :P + n]), ref["score"], dtype, "score")
            if lse is not None:
                assert_close(to_host(lse[b:b + 1, :, :n]), ref["lse"], dtype, "lse")
        assert (out[b, :, n:] == 5.0).all()  # rows beyond the sequence are left alone
