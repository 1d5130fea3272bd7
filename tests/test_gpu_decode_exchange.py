"""Divided generation steps at the sizes from which a (batch, head) is divided, and with numbers of pairs that the XCDs do not share
out evenly (the launch is padded to eight)."""
import pytest

from test_gpu_decode import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,B,H,rows", [
    ("bf16", 128, 1, 8, 478), ("bf16", 128, 1, 8, 479),     # 240 KB, eight shares
    ("f32", 128, 1, 32, 238), ("f32", 128, 1, 32, 239),
    ("bf16", 128, 2, 32, 638), ("bf16", 128, 2, 32, 639),   # 320 KB, four
    ("bf16", 128, 1, 4, 3070), ("bf16", 128, 1, 4, 3071),   # 1.5 MB, eight and sixteen
    ("bf16", 64, 3, 11, 1500),                              # 33 pairs: 40 a share, six shares
    ("f32", 64, 1, 1, 2000), ("bf16", 128, 5, 17, 700),     # 1 and 85
])
def test_divided_launch_sizes(dtype, D, B, H, rows):
    for victim in (rows - 25, 0):
        _case(dtype, D, B, H, 1, rows + 2, rows, victim, seed=rows + victim)
