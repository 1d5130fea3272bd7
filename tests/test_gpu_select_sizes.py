"""Anchor choice at the sizes where the kernel's shape changes, over ranges of scores from one value to all of fp32."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_18121_amd import binding as ec

pytestmark = pytest.mark.gpu


def _scores(kind, G, T, rng):
    if kind == "equal":
        return np.full((1, G, T), 0.25, np.float32)
    if kind == "few values":      # ties at every threshold
        return rng.integers(-3, 4, (1, G, T)).astype(np.float32)
    if kind == "one bit":         # keys that differ in their lowest bit only
        return (np.full((1, G, T), 1.0, np.float32).view(np.int32) + rng.integers(0, 2, (1, G, T), dtype=np.int32)).view(np.float32)
    if kind == "all":             # every bit of the keys counts: both signs, subnormals, infinities
        s = rng.integers(0, 1 << 32, (1, G, T), dtype=np.uint64).astype(np.uint32).view(np.float32)
        return np.where(np.isnan(s), np.float32(np.inf), s)
    s = np.log((T + 1.0) / (np.arange(T) + 1.0)) * np.exp(0.1 * rng.standard_normal((1, G, T)))
    return s.astype(np.float32)


@pytest.mark.parametrize("kind", ["equal", "few values", "one bit", "all", "prompt"])
@pytest.mark.parametrize("T", [1, 5, 64, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193])
def test_sizes(T, kind):
    rng = np.random.default_rng(T)
    s = _scores(kind, 3, T, rng)   # three groups: rows of odd T do not start on 16-byte boundaries
    for n in sorted({1, max(1, T // 3), max(1, T - 1), T}):
        first, last = (0, 0) if n < 2 else (1, 1)
        got = torch.zeros((1, 3, n), dtype=torch.int32, device="cuda")
        ec.ec_select_anchors(torch.from_numpy(s).cuda(), n, first, last, got)
        np.testing.assert_array_equal(got.cpu().numpy(), oracle.select_anchors(s.astype(np.float64), n, first, last))
