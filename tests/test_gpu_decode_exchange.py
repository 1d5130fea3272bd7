"""Divided generation steps at the sizes from which a (batch, head) is divided, and with numbers of pairs that the XCDs do not share
out evenly (the launch is padded to eight)."""
import pytest

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
