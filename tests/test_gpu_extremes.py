"""Scoring calls whose scores are infinite, enormous or not numbers: every launch shape gives the softmax that remains.
References: the same in 64 bits, where the products do not overflow."""
import numpy as np
import pytest
import torch

from paper_2407_18121_amd import binding as ec
from util import assert_close, to_host, torch_dtype

pytestmark = pytest.mark.gpu

# (dtype, heads, rows) of every launch shape at D = 64
SHAPES = [
    ("f32", 2, 200), ("f32", 32, 200), ("f32", 128, 200),     # four, two, one wave(s) on the keys of 16 queries
    ("bf16", 130, 200), ("bf16", 2, 200), ("bf16", 2, 300),   # single tiles; the same, two groups in the column pass
    ("bf16", 2, 1100), ("bf16", 128, 900),                    # two groups in both passes; pairs in both
]


def _inputs(H, T, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((1, H, T, 64), generator=g) for _ in range(3)]


def _score(q, k, v, dtype, scale):
    q, k, v = (x.to(torch_dtype(dtype)).cuda() for x in (q, k, v))
    B, H, T, D = q.shape
    out, lse = torch.zeros_like(q), torch.zeros((B, H, T), device="cuda")
    score = torch.zeros((B, H, T), device="cuda")
    ec.ec_prefill_score(q, k, v, out, lse, score, scale, ec.new_workspace(ec.EC_FN_PREFILL_SCORE, B, H, T, D, ec.dtype_code(q)))
    torch.cuda.synchronize()
    return to_host(out), to_host(lse), to_host(score)


def _reference(q, k, v, dtype, scale, P=0):
    q, k, v = (x.to(torch_dtype(dtype)).double() for x in (q, k, v))
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) * scale
    s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool).triu(1 + P), -torch.inf)
    a = torch.softmax(s, -1)
    return torch.matmul(a, v).numpy(), torch.logsumexp(s, -1).numpy(), a.sum(-2).numpy()


@pytest.mark.parametrize("dtype,H,T", SHAPES)
def test_first_keys_at_minus_infinity(dtype, H, T):
    """Most queries score the first 70 keys -inf: more than any kernel's first tile, which leaves them without a maximum."""
    q, k, v = _inputs(H, T, 1)
    q[..., 0] = k[..., 0] = 0.0
    q[:, :, 70:, 0], k[:, :, :70, 0] = 1e30, -1e30
    got, ref = _score(q, k, v, dtype, 0.125), _reference(q, k, v, dtype, 0.125)
    for name, x, y in zip(("out", "lse", "score"), got, ref):
        assert_close(x, y, dtype, name)


@pytest.mark.parametrize("magnitude", [-1e33, -1e12, 1e12, 1e33])
@pytest.mark.parametrize("H,T", [(H, T) for dtype, H, T in SHAPES if dtype == "f32"])
def test_enormous_fp32_scores(H, T, magnitude):
    """Scores so far apart that one key takes it all.  (The column sums are not compared: they subtract a stored log-sum-exp
    whose own rounding is many orders above one.)"""
    q, k, v = _inputs(H, T, 2)
    q[..., 0] = magnitude
    g = torch.Generator().manual_seed(3)
    rank = torch.stack([torch.randperm(T, generator=g) for _ in range(H)])[None]
    k[..., 0] = 1.0 + rank / T
    out, lse, _ = _score(q, k, v, "f32", 0.125)
    ref_out, ref_lse, _ = _reference(q, k, v, "f32", 0.125)
    assert_close(out, ref_out, "f32", "out")
    np.testing.assert_allclose(lse, ref_lse, rtol=1e-6)  # a product, a sum and two scalings in 24 bits


@pytest.mark.parametrize("dtype,H,T", SHAPES)
@pytest.mark.parametrize("what", ["a query of NaN", "a query whose scores are all -inf"])
def test_a_query_without_a_softmax_stays_among_the_keys_it_sees(dtype, H, T, what):
    """Column sums of keys behind the query, and the output rows of all others, are what they are without it."""
    q, k, v = _inputs(H, T, 4)
    q[..., 0], k[..., 0] = 0.0, -1e30
    where = sorted({37, 64, 101, 131, T - 30} & set(range(T)))   # inside, at the start of and late in a block of keys
    ref_out, ref_lse, _ = _reference(q, k, v, dtype, 0.125)
    for m in where:
        bad = q.clone()
        if what == "a query of NaN":
            bad[:, :, m] = torch.nan
        else:
            bad[:, :, m, 0] = 1e30
        out, lse, score = _score(bad, k, v, dtype, 0.125)
        others = [i for i in range(T) if i != m]
        assert_close(out[:, :, others], ref_out[:, :, others], dtype, "out")
        assert_close(lse[:, :, others], ref_lse[:, :, others], dtype, "lse")
        ref = _reference(q[:, :, m + 1:], k, v, dtype, 0.125, m + 1)[2]
        assert_close(score[:, :, m + 1:], ref[:, :, m + 1:], dtype, "score")
        assert np.isnan(score[:, :, :m + 1]).all() and np.isnan(out[:, :, m]).all()
