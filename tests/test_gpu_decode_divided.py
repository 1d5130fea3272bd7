"""Generation steps whose (batch, head) pairs are divided over several workgroups, and the launch shapes around them."""
import math

import pytest
import torch

from paper_2407_18121_amd import binding as ec
from test_gpu_decode import _case

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _step(dtype, D, B, H, rows, victim, seed=0, **shape):
    """One step on device tensors; (out, k_cache, v_cache, pos)."""
    torch.manual_seed(seed)
    t = lambda *s: torch.randn(*s, device="cuda").to(DT[dtype])
    q, kn, vn, kc, vc = t(B, H, D), t(B, H, D), t(B, H, D), t(B, H, rows + 2, D), t(B, H, rows + 2, D)
    out, pos = torch.zeros_like(q), torch.arange(rows + 2, dtype=torch.int32, device="cuda").repeat(B, 1, 1)
    ws = torch.zeros(4 * B * H * 64 * (D + 2), dtype=torch.uint8, device="cuda")
    ec.ec_decode_step_shaped(q, kn, vn, kc, vc, pos, rows, victim, 7, D ** -0.5, out, ws, **shape)
    return out, kc, vc, pos


# on both sides of the size from which a pair is divided (256 KB in bf16 D128, else 240; 340 for 64 pairs), and every place
# the victim can have: in the owner's registers, in its share, in a helper's share, the first row, the new row, none
@pytest.mark.parametrize("dtype,D,B,H,rows", [("bf16", 128, 1, 8, 510), ("bf16", 128, 1, 8, 511), ("bf16", 64, 2, 8, 958),
                                              ("bf16", 64, 2, 8, 959), ("f32", 128, 1, 8, 238), ("f32", 128, 1, 8, 239),
                                              ("bf16", 128, 2, 32, 678), ("bf16", 128, 2, 32, 679),
                                              ("bf16", 128, 1, 8, 574), ("bf16", 128, 1, 8, 575), ("bf16", 64, 2, 8, 1151),
                                              ("f32", 128, 1, 8, 287), ("f32", 64, 1, 5, 2100), ("bf16", 128, 2, 32, 703)])
def test_divided_step(dtype, D, B, H, rows):
    for victim in (-1, rows - 25, rows - 90, rows // 2, 0, rows):
        _case(dtype, D, B, H, 1, rows + 2, rows, victim, seed=rows + victim)


@pytest.mark.parametrize("scale", [1e-3, 1.0, 37.5])
def test_divided_step_scales(scale):
    _case("bf16", 128, 1, 8, 1, 702, 700, 675, seed=5, scale=scale)


def test_divided_step_ragged():
    """Sequences of one launch on both sides of one share, and an empty one."""
    B, H, D, cap = 5, 8, 128, 1300
    lens, victims = [1290, 0, 90, 600, 191], [1265, -1, 65, 0, 191]
    torch.manual_seed(3)
    q, kn, vn = (torch.randn(B, H, D, device="cuda").bfloat16() for _ in range(3))
    kc, vc = (torch.randn(B, H, cap, D, device="cuda").bfloat16() for _ in range(2))
    pos, out = torch.arange(cap, dtype=torch.int32, device="cuda").repeat(B, 1, 1), torch.zeros_like(q)
    want = [x.clone() for x in (kc, vc, pos, out)]
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    ec.ec_decode_step_varlen(q, kn, vn, kc, vc, pos, i32(lens), i32(victims), i32([9] * B), 0.088, out)
    for b in range(B):
        one = [x[b:b + 1].contiguous() for x in (q, kn, vn, *want)]
        ec.ec_decode_step_shaped(*one[:6], lens[b], victims[b], 9, 0.088, one[6], None, waves=4, splits=1)
        for got, ref in zip((kc, vc, pos), one[3:6]):
            assert torch.equal(got[b:b + 1], ref)
        # the same sums in another order: fp32 rounding, then one rounding to bf16 that may fall to the other side
        torch.testing.assert_close(out[b:b + 1].float(), one[6].float(), rtol=2 ** -7, atol=1e-5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_lines_that_are_taken(dtype):
    """More shares than there are lines, and launches on two streams whose output rows share lines: whoever finds its line
    taken, or its helper not there yet, forms the share itself, with the same result bit for bit."""
    D, rows = 64, 900
    want = _step(dtype, D, 1, 8, rows, rows // 3, waves=4, splits=16)
    many = _step(dtype, D, 16, 24, 200, 40, waves=2, splits=64)  # 24192 shares, 256 lines of each XCD
    again = _step(dtype, D, 16, 24, 200, 40, waves=2, splits=64)
    plain = _step(dtype, D, 16, 24, 200, 40, waves=2, splits=1)
    for a, b, c in zip(many, again, plain):
        assert torch.equal(a, b)
        # in another order: rounding of a 64-term product and 200-term sum in fp32, and of bf16 once
        torch.testing.assert_close(a.float(), c.float(), rtol=2 ** -7 if dtype == "bf16" else 1e-5, atol=1e-5)
    streams = [torch.cuda.Stream() for _ in range(4)]
    got = []
    for i in range(12):
        with torch.cuda.stream(streams[i % 4]):
            got.append(_step(dtype, D, 1, 8, rows, rows // 3, waves=4, splits=16))
    torch.cuda.synchronize()
    for g in got:
        assert all(torch.equal(a, b) for a, b in zip(g, want))


# the victim is the last row of share 1 while the rows behind it, share 0, all fit into the owner's registers; in the first line
# there are more shares than lines, so that owners form share 1 themselves, after share 0
@pytest.mark.parametrize("dtype,D,B,H,rows,waves,splits", [
    ("bf16", 64, 16, 24, 200, 2, 64), ("f32", 64, 16, 24, 200, 2, 64), ("bf16", 128, 1, 8, 640, 8, 8), ("bf16", 128, 1, 4, 640, 8, 16),
    ("f32", 128, 1, 8, 399, 4, 16), ("bf16", 64, 2, 3, 700, 4, 16), ("bf16", 128, 2, 4, 390, 4, 16)])
def test_victim_is_the_last_row_of_the_next_share(dtype, D, B, H, rows, waves, splits):
    share = -(-(rows + 1) // splits)
    first = rows + 1 - share                          # of share 0
    for victim in (first - 1, first, first - 2):
        _case(dtype, D, B, H, 1, rows + 2, rows, victim, seed=rows + victim, shape=(waves, 4, splits))
    _case(dtype, D, B, H, 1, rows + 2, rows, first - 1, seed=rows, shape=(waves, 4, 1))


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_long_caches_of_large_batches(dtype, D):
    """The shape with one tile in flight does the same sums in the same order as the deep one of its width."""
    row = 2 * D * (2 if dtype == "bf16" else 4)
    for B, H in ((9, 29), (16, 32)):
        rows = (320 << 10) // row + 3
        a = _step(dtype, D, B, H, rows, rows - 25)
        waves = 2 if dtype == "bf16" and B * H >= 512 else 4
        for x, y in zip(a, _step(dtype, D, B, H, rows, rows - 25, waves=waves, splits=1)):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [60, 1300])
def test_scores_that_are_not_finite(dtype, rows):
    """Heads with rows of score -inf (left out), of score +inf or NaN (the head's output is NaN), with an infinite V row, and a
    whole head of -inf; others stay as they are."""
    B, H, D = 1, 8, 64
    torch.manual_seed(11)
    t = lambda *s: torch.randn(*s, device="cuda").to(DT[dtype])
    q, kn, vn, kc, vc = t(B, H, D), t(B, H, D), t(B, H, D), t(B, H, rows + 1, D), t(B, H, rows + 1, D)
    sign = torch.where(q[0, :, 0] > 0, 1.0, -1.0)
    kc[0, 1, ::3, 0] = -math.inf * sign[1]
    kc[0, 2, rows // 2, 0] = math.inf * sign[2]
    kc[0, 3, 5, 7] = math.nan
    vc[0, 4, rows - 2, 3] = math.inf
    kc[0, 5, :, 0] = -math.inf * sign[5]
    kn[0, 5, 0] = -math.inf * sign[5]
    k, v = kc.double().clone(), vc.double().clone()
    k[:, :, rows], v[:, :, rows] = kn.double(), vn.double()
    s = (k * q.double()[:, :, None]).sum(-1) * D ** -0.5
    w = torch.softmax(s, -1)[..., None]
    want = torch.where((w == 0) & ~v.isnan(), torch.zeros_like(v), w * v).sum(-2).float()
    out = torch.zeros_like(q)
    ec.ec_decode_step(q, kn, vn, kc, vc, None, rows, -1, 0, D ** -0.5, out, None, G=1)
    # a bf16 value is rounded once; fp32 sums of up to 1301 terms
    torch.testing.assert_close(out.float(), want, rtol=2 ** -7 if dtype == "bf16" else 1e-4, atol=1e-4, equal_nan=True)


@pytest.mark.parametrize("dtype,D,rows", [("bf16", 128, 700), ("f32", 64, 800)])
def test_frequency_step_divided(dtype, D, rows):
    """One sequence (divided) against the same one among 20 (not divided): masses, outputs and caches."""
    H = 8
    torch.manual_seed(2)
    t = lambda *s: torch.randn(*s, device="cuda").to(DT[dtype])
    one = [t(1, H, D), t(1, H, D), t(1, H, D), t(1, H, rows + 2, D), t(1, H, rows + 2, D)]
    res = []
    for B in (1, 20):
        q, kn, vn, kc, vc = (x.repeat(B, 1, *([1] * (x.dim() - 2))) for x in one)
        out, freq = torch.zeros_like(q), torch.ones(B, 1, rows + 2, device="cuda")
        ws = ec.new_workspace(ec.EC_FN_DECODE_SCORE_STEP, B, H, rows + 2, D, ec.dtype_code(kc))
        ec.ec_decode_score_step(q, kn, vn, kc, vc, None, freq, rows, 3, D ** -0.5, out, ws)
        res.append((out, kc, vc, freq))
    for x, y in zip(*res):
        # the divided sums in another order: fp32 rounding, then one of bf16
        torch.testing.assert_close(y, x.expand_as(y).contiguous(), rtol=2 ** -7 if x.dtype == torch.bfloat16 else 1e-5, atol=1e-6)


@pytest.mark.parametrize("dtype,D,rows", [("bf16", 128, 700), ("f32", 64, 1200)])
def test_launches_that_share_a_throw_away_output(dtype, D, rows):
    """Divided frequency steps of four streams over caches of their own, all with one output that nobody reads: the masses are
    those of each launch alone."""
    H, streams = 8, [torch.cuda.Stream() for _ in range(4)]
    t = lambda *s: torch.randn(*s, device="cuda").to(DT[dtype])
    out = torch.zeros(1, H, D, device="cuda", dtype=DT[dtype])

    def step(inputs, out):
        q, kn, vn, kc, vc = inputs
        freq = torch.zeros(1, H, rows + 1, device="cuda")
        ws = ec.new_workspace(ec.EC_FN_DECODE_SCORE_STEP, 1, H, rows + 1, D, ec.dtype_code(kc))
        ec.ec_decode_score_step(q, kn, vn, kc.clone(), vc.clone(), None, freq, rows, 3, D ** -0.5, out, ws)
        return freq, ws
    torch.manual_seed(4)
    cases = [(t(1, H, D), t(1, H, D), t(1, H, D), t(1, H, rows + 1, D), t(1, H, rows + 1, D)) for _ in streams]
    want = [step(c, torch.zeros_like(out))[0] for c in cases]
    torch.cuda.synchronize()
    got = []
    for _ in range(8):
        for i, stream in enumerate(streams):
            with torch.cuda.stream(stream):
                got.append((i, step(cases[i], out)))
    torch.cuda.synchronize()
    for i, (freq, _) in got:
        assert torch.equal(freq, want[i])
