"""Generation steps in every launch shape that the library chooses by itself, through the ordinary calls, and at the ends of the
numbers' range, against the same step in 64 bits (softmax, append and removal written out in torch)."""
import pytest
import torch

from paper_2407_18121_amd import binding as ec

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "bf16": torch.bfloat16}
KIB = 1 << 10


def _rows(dtype, D, kib):
    """Rows, the new one included, whose K and V take `kib` KiB."""
    return kib * KIB // (2 * D * (2 if dtype == "bf16" else 4))


def _inputs(dtype, D, B, H, cap, seed, shift=0):
    """q, k_new, v_new, k_cache, v_cache; `shift` elements behind an allocation's start."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def t(*shape):
        x = torch.randn(shape, device="cuda", generator=g).to(DT[dtype])
        flat = torch.empty(x.numel() + shift, device="cuda", dtype=DT[dtype])[shift:]
        return flat.copy_(x.flatten()).view(shape)
    return t(B, H, D), t(B, H, D), t(B, H, D), t(B, H, cap, D), t(B, H, cap, D)


def _expect(q, kn, vn, kc, vc, n, victim, scale):
    """(out, cache rows afterwards, softmax) of [B,H] pairs with n cached rows."""
    k, v = (torch.cat([c[:, :, :n], x[:, :, None]], 2) for c, x in ((kc, kn), (vc, vn)))
    s = (k.double() * q.double()[:, :, None]).sum(-1) * scale
    p = (s - s.amax(-1, keepdim=True)).exp()  # torch.softmax on the device gives zero for what is subnormal in fp32
    p = p / p.sum(-1, keepdim=True)
    out = (p[..., None] * v.double()).sum(2)
    if victim >= 0:
        k, v = (torch.cat([x[:, :, :victim], x[:, :, victim + 1:]], 2) for x in (k, v))
    return out, k, v, p


def _close(got, want, dtype):
    # one rounding to bf16, half a unit of the value; fp32: sums of up to some thousand terms of size one
    torch.testing.assert_close(got.double(), want, rtol=2 ** -8 if dtype == "bf16" else 1e-5, atol=1e-5)


# (type, D, pairs, KiB of K and V of one pair): each side of every line of the rule
EDGES = [("bf16", 64, 8, 32, 319), ("bf16", 64, 8, 33, 320), ("bf16", 64, 16, 32, 319), ("bf16", 64, 16, 32, 320),
         ("bf16", 64, 32, 32, 79), ("bf16", 64, 32, 32, 80), ("bf16", 64, 32, 44, 110),
         ("bf16", 128, 8, 33, 32), ("bf16", 128, 8, 33, 33), ("bf16", 128, 8, 33, 320), ("bf16", 128, 16, 32, 159),
         ("bf16", 128, 16, 32, 160), ("bf16", 128, 32, 32, 79), ("bf16", 128, 32, 32, 80), ("bf16", 128, 32, 44, 109),
         ("bf16", 128, 32, 44, 110),
         ("f32", 128, 8, 33, 139), ("f32", 128, 8, 33, 140), ("f32", 128, 32, 32, 139), ("f32", 128, 32, 32, 140),
         ("f32", 128, 32, 32, 300), ("f32", 128, 32, 44, 199), ("f32", 128, 32, 44, 200), ("f32", 64, 16, 32, 320), ("f32", 64, 32, 32, 33),
         ("f32", 64, 32, 44, 110)]


@pytest.mark.parametrize("dtype,D,B,H,kib", EDGES)
def test_step(dtype, D, B, H, kib):
    n = _rows(dtype, D, kib) - 1
    for victim in (-1, n - 25, n // 3, 0, n):
        q, kn, vn, kc, vc = _inputs(dtype, D, B, H, n + 2, n + victim)
        out, k, v, _ = _expect(q, kn, vn, kc, vc, n, victim, D ** -0.5)
        got, beyond = torch.zeros_like(q), kc[:, :, n + 1].clone()
        pos = torch.arange(n + 2, dtype=torch.int32, device="cuda").repeat(B, 1, 1)
        ec.ec_decode_step(q, kn, vn, kc, vc, pos, n, victim, 77, D ** -0.5, got, None)
        _close(got, out, dtype)
        m = k.shape[2]
        assert torch.equal(kc[:, :, :m], k) and torch.equal(vc[:, :, :m], v) and torch.equal(kc[:, :, n + 1], beyond)
        want = torch.cat([torch.arange(n), torch.tensor([77])])
        assert torch.equal(pos[0, 0, :m].cpu().long(), want[torch.arange(n + 1) != victim])


@pytest.mark.parametrize("dtype,D,B,H,kib", [e for e in EDGES if e[4] < 300] + [
    ("bf16", 64, 32, 32, 107), ("bf16", 64, 44, 32, 107), ("bf16", 128, 44, 32, 147), ("bf16", 128, 16, 32, 400), ("bf16", 128, 32, 32, 107),
    ("f32", 128, 32, 32, 187), ("f32", 128, 44, 32, 267), ("f32", 128, 32, 32, 400)])
def test_step_of_a_ragged_batch(dtype, D, B, H, kib):
    """Sequences of half to all of the buffer, an empty one and one of a single row."""
    cap = _rows(dtype, D, kib)
    lens = [cap - 1, 0, 1] + [cap // 2 + (7 * b) % (cap - cap // 2) for b in range(B - 3)]
    victims = [(-1, n - min(n, 25), n // 3, 0, n)[b % 5] for b, n in enumerate(lens)]
    q, kn, vn, kc, vc = _inputs(dtype, D, B, H, cap, kib)
    want = [_expect(q[b:b + 1], kn[b:b + 1], vn[b:b + 1], kc[b:b + 1], vc[b:b + 1], lens[b], victims[b], D ** -0.5)
            for b in range(B)]
    got = torch.zeros_like(q)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    ec.ec_decode_step_varlen(q, kn, vn, kc, vc, None, i32(lens), i32(victims), None, D ** -0.5, got, G=1)
    for b, (out, k, v, _) in enumerate(want):
        _close(got[b:b + 1], out, dtype)
        m = k.shape[2]
        assert torch.equal(kc[b:b + 1, :, :m], k) and torch.equal(vc[b:b + 1, :, :m], v)


@pytest.mark.parametrize("dtype,D,B,H,kib", EDGES + [("bf16", 128, 2, 40, 200), ("f32", 64, 1, 8, 400)])
@pytest.mark.parametrize("groups", ["layer", "head"])
def test_frequency_step(dtype, D, B, H, kib, groups):
    """Masses and output of the frequency policy's step: its kernels store a score per row."""
    n, G = _rows(dtype, D, kib) - 1, 1 if groups == "layer" else H
    q, kn, vn, kc, vc = _inputs(dtype, D, B, H, n + 2, n)
    out, k, v, p = _expect(q, kn, vn, kc, vc, n, -1, D ** -0.5)
    freq = torch.rand(B, G, n + 2, device="cuda")
    want = freq.double()
    want[:, :, n] = 0
    want[:, :, :n + 1] += p.mean(1, keepdim=True) if G == 1 else p
    got = torch.zeros_like(q)
    ws = ec.new_workspace(ec.EC_FN_DECODE_SCORE_STEP, B, H, n + 2, D, ec.dtype_code(kc))
    ec.ec_decode_score_step(q, kn, vn, kc, vc, None, freq, n, 5, D ** -0.5, got, ws)
    _close(got, out, dtype)
    assert torch.equal(kc[:, :, :n + 1], k) and torch.equal(vc[:, :, :n + 1], v)
    # a probability of at most one and a mass of the same size, in fp32
    torch.testing.assert_close(freq.double(), want, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("B,H,n", [(1, 8, 37), (1, 8, 1300), (9, 32, 150), (44, 32, 90)])
def test_tensors_that_start_at_any_element(dtype, D, B, H, n):
    q, kn, vn, kc, vc = _inputs(dtype, D, B, H, n + 1, n, shift=1)
    out, k, v, _ = _expect(q, kn, vn, kc, vc, n, n - 25, D ** -0.5)
    got = torch.zeros_like(q)
    ec.ec_decode_step(q, kn, vn, kc, vc, None, n, n - 25, 5, D ** -0.5, got, None, G=1)
    _close(got, out, dtype)
    assert torch.equal(kc[:, :, :n], k) and torch.equal(vc[:, :, :n], v)


RANGES = {  # exponents of keys and of queries, scale
    "keys below the normal range": (-130, 123, 1.0),
    "queries below the normal range": (125, -130, 0.0884),
    "queries that scaling takes below it": (124, -124, 0.0884),
    "large queries": (-128, 127, 1.0),
    "large keys": (127, -128, 1.0),
}


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("n", [40, 1300])
@pytest.mark.parametrize("what", RANGES)
def test_queries_and_keys_at_the_ends_of_the_range(dtype, D, n, what):
    """The scores are of size one; neither their products nor their sums leave the range that q * scale stays in."""
    at_k, at_q, scale = RANGES[what]
    q, kn, vn, kc, vc = _inputs(dtype, D, 2, 8, n + 1, n)
    scaled = lambda x, e: (x.double().clamp(-1.3, 1.3) * 2.0 ** e).to(x.dtype)
    q, kn, kc = scaled(q, at_q), scaled(kn, at_k), scaled(kc, at_k)
    out, *_ = _expect(q, kn, vn, kc, vc, n, -1, scale)
    got = torch.zeros_like(q)
    ec.ec_decode_step(q, kn, vn, kc, vc, None, n, -1, 5, scale, got, None, G=1)
    _close(got, out, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_near_the_largest_number(dtype):
    """Scores of 2.7e38 in base-2 units: the unscaled half of one would still fit, twice one would not."""
    n, D = 40, 64
    q, kn, vn, kc, vc = _inputs(dtype, D, 1, 4, n + 1, 1)
    q[..., 0], kc[..., 0], kn[..., 0] = 2.0 ** 126, 1.0, 1.0
    kc[:, :, 7:9, 0] = 2.203125
    out, *_ = _expect(q, kn, vn, kc, vc, n, -1, 1.0)
    got = torch.zeros_like(q)
    ec.ec_decode_step(q, kn, vn, kc, vc, None, n, -1, 5, 1.0, got, None, G=1)
    _close(got, out, dtype)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("where", ["beside the largest", "behind it", "before it", "in another share"])
def test_weights_below_the_normal_range(dtype, D, where):
    """The row of the largest score has no V; all the others weigh 2^-127 to 2^-131 and have V rows of 1e34 and more."""
    H, n = 8, 1300 if where == "in another share" else 300
    q, kn, vn, kc, vc = _inputs(dtype, D, 1, H, n + 1, n)
    at = {"beside the largest": 150, "behind it": 0, "before it": n - 1, "in another share": n // 2}[where]
    for x in (q, kn, kc):
        x.zero_()
    low = lambda x: -88.5 - 2 * torch.rand(x.shape[:-1], device="cuda")
    q[..., 0], kn[..., 0], kc[..., 0] = 1.0, low(kn), low(kc)
    for x in (vn, vc):
        x.copy_(1e34 * (1 + x.double().abs().clamp(max=2)))
    kc[:, :, at], vc[:, :, at] = 0, 0
    out, *_ = _expect(q, kn, vn, kc, vc, n, -1, 1.0)
    got = torch.zeros_like(q)
    ec.ec_decode_step(q, kn, vn, kc, vc, None, n, -1, 5, 1.0, got, None, G=1)
    # scores of up to 131 in base-2 units, three roundings of 2^-24 each, are exponents: 131 * 3 * 2^-24 * ln 2 < 2^-15
    torch.testing.assert_close(got.double(), out, rtol=2 ** -8 + 2 ** -15 if dtype == "bf16" else 2 ** -15, atol=0)
