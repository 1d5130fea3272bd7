"""Divided generation steps at the sizes from which a (batch, head) is divided, and with numbers of pairs that the XCDs do not share
out evenly (the launch is padded to eight)."""
import pytest
import torch

from paper_2407_18121_amd import binding as ec
from paper_2407_18121_amd.tune import graph_time_ms
from test_gpu_decode import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,B,H,rows", [
    ("bf16", 128, 1, 8, 478), ("bf16", 128, 1, 8, 479),     # one workgroup each
    ("bf16", 128, 1, 8, 510), ("bf16", 128, 1, 8, 511),     # 256 KB: one workgroup; six shares, of at least 48 KB each
    ("f32", 128, 1, 32, 238), ("f32", 128, 1, 32, 239),     # 240 KB: one, five
    ("bf16", 128, 1, 48, 583), ("bf16", 128, 8, 10, 775),   # 292 KB, five shares; 388 KB, three
    ("bf16", 128, 2, 32, 678), ("bf16", 128, 2, 32, 679),   # 340 KB, four
    ("bf16", 128, 1, 4, 3070), ("bf16", 128, 1, 4, 3071),   # 1.5 MB, eight and sixteen
    ("bf16", 64, 3, 11, 1500),                              # 33 pairs: 40 workgroups a share, six shares
    ("bf16", 64, 1, 17, 8200), ("bf16", 128, 4, 7, 3100),   # 17 and 28 pairs of 2 and 1.5 MB: eight
    ("f32", 64, 1, 1, 2000), ("bf16", 128, 5, 17, 700), ("bf16", 128, 5, 17, 1030),  # 1 and 85: eight, one (below 435 KB) and two
])
def test_divided_launch_sizes(dtype, D, B, H, rows):
    for victim in (rows - 25, 0):
        _case(dtype, D, B, H, 1, rows + 2, rows, victim, seed=rows + victim)


def _timer(H, rows, D=128):
    """us(splits) of a launch of one sequence."""
    t = lambda *s: torch.randn(*s, device="cuda").bfloat16()
    q, kn, vn, kc, vc = t(1, H, D), t(1, H, D), t(1, H, D), t(1, H, rows + 2, D), t(1, H, rows + 2, D)
    out, ws = torch.empty_like(q), torch.zeros(4 * H * 64 * (D + 2), dtype=torch.uint8, device="cuda")

    def us(splits):
        step = lambda: ec.ec_decode_step_shaped(q, kn, vn, kc, vc, None, rows, rows - 25, 7, 0.1, out, ws, waves=4, unroll=4, splits=splits, G=1)
        return min(graph_time_ms(lambda: [step() for _ in range(16)]) for _ in range(3)) / 16 * 1e3
    return us


@pytest.mark.parametrize("H,splits", [(8, 8), (8, 16), (16, 16), (16, 33), (32, 8), (32, 33), (24, 64)])
def test_shares_come_from_their_helpers(H, splits):
    """Owners that never met a helper would form every share themselves, with the same bits, in the time of one workgroup or more: a
    divided launch has to be faster than that.  Measured 11 to 24 us against 40 to 43; with 33 and 64 shares, where pairs of an XCD that
    wanted the same lines took 99 to 153, most of an XCD's lines are in use."""
    us = _timer(H, 4400)
    assert us(splits) < 0.8 * us(1)


def test_owners_do_not_wait_for_helpers_without_a_place():
    """Launches of many more workgroups than fit: helpers start when owners have left, which form the shares themselves.  Measured 2.4
    times the undivided launch, with an owner that looks for its helper 24 times 3.7."""
    us = _timer(1536, 150)
    assert us(2) < 3 * us(1)
