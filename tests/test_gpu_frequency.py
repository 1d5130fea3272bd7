"""GPU parity: the "Frequency" discard policy of the generation stage (Sec. 4.1 Baselines, Frequency Cache;
ablation Table 3a) -- ec_decode_score_step and ec_evict_min vs the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_18121_amd import binding as ec
from util import assert_close, quantize, to_dev, to_host, torch_dtype

pytestmark = pytest.mark.gpu


def _cache(rng, B, H, cap, n, D, dtype):
    kc = np.zeros((B, H, cap, D), np.float32)
    vc = np.zeros((B, H, cap, D), np.float32)
    kc[:, :, :n] = quantize(rng.standard_normal((B, H, n, D)) * 1.5, dtype)
    vc[:, :, :n] = quantize(rng.standard_normal((B, H, n, D)), dtype)
    if n > 0:
        kc[:, :, 0] = quantize(kc[:, :, 0] * 6, dtype)
    return kc, vc


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("B,H,Gmode,cap,cache_len", [
    (1, 2, "layer", 8, 0), (2, 3, "head", 40, 5), (2, 3, "layer", 70, 64), (1, 4, "layer", 300, 257),
    (3, 2, "head", 700, 655), (2, 2, "layer", 1100, 1029),
])
def test_decode_score_step_parity(dtype, D, B, H, Gmode, cap, cache_len):
    rng = np.random.default_rng(cap * 7 + cache_len + D)
    G = 1 if Gmode == "layer" else H
    scale = 1.0 / np.sqrt(D)
    kc, vc = _cache(rng, B, H, cap, cache_len, D, dtype)
    q, kn, vn = (quantize(rng.standard_normal((B, H, D)), dtype) for _ in range(3))
    pos = np.tile(np.arange(cap, dtype=np.int32) * 3 + 1, (B, G, 1))
    pos[:, :, cache_len:] = -7
    freq = (rng.random((B, G, cap)) * 5).astype(np.float32)
    freq[:, :, cache_len:] = 77.0                        # stale values beyond the cache: the new row is SET

    okc, ovc, opos, ofreq = kc.astype(np.float64), vc.astype(np.float64), pos.copy(), freq.astype(np.float64)
    oout, _ = oracle.decode_score_step(q, kn, vn, okc, ovc, opos, ofreq, cache_len, 4242, scale)

    dkc, dvc, dpos, dfreq = to_dev(kc, dtype), to_dev(vc, dtype), torch.from_numpy(pos).cuda(), torch.from_numpy(freq).cuda()
    dout = torch.full((B, H, D), float("nan"), dtype=torch_dtype(dtype), device="cuda")
    ws = ec.new_workspace(ec.EC_FN_DECODE_SCORE_STEP, B, H, cap, D, ec.dtype_code(dkc))
    ec.ec_decode_score_step(to_dev(q, dtype), to_dev(kn, dtype), to_dev(vn, dtype), dkc, dvc, dpos, dfreq, cache_len,
                            4242, scale, dout, ws)
    torch.cuda.synchronize()
    n = cache_len + 1
    assert_close(to_host(dout), oout, dtype, "out")
    # masses are probabilities added to O(1) counts: the fp32 bar applies whatever the storage type
    got = dfreq.cpu().numpy().astype(np.float64)
    assert np.abs(got[:, :, :n] - ofreq[:, :, :n]).max() <= (1e-4 if dtype == "f32" else 2e-3)
    assert (got[:, :, n:] == 77.0).all()
    np.testing.assert_array_equal(to_host(dkc)[:, :, :n], okc[:, :, :n])
    np.testing.assert_array_equal(to_host(dvc)[:, :, :n], ovc[:, :, :n])
    np.testing.assert_array_equal(dpos.cpu().numpy(), opos)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("B,H,Gmode,cap,length,pf,pr", [
    (1, 2, "layer", 8, 3, 1, 1),        # a single candidate
    (2, 3, "head", 40, 17, 1, 1), (2, 3, "layer", 70, 65, 0, 2), (1, 4, "layer", 300, 258, 1, 25),
    (3, 2, "head", 700, 656, 4, 1), (2, 2, "layer", 1100, 1100, 1, 1), (1, 2, "layer", 5000, 4999, 1, 1),
])
def test_evict_min_bit_exact(dtype, D, B, H, Gmode, cap, length, pf, pr):
    rng = np.random.default_rng(cap * 11 + length + D)
    G = 1 if Gmode == "layer" else H
    kc, vc = _cache(rng, B, H, cap, length, D, dtype)
    pos = np.tile(np.arange(cap, dtype=np.int32) * 3 + 1, (B, G, 1))
    freq = (np.round(rng.random((B, G, cap)) * 64) / 64).astype(np.float32)   # plenty of exact ties
    freq[0, 0, 0] = -5.0                                   # protected rows are never taken
    freq[0, 0, length - 1] = -5.0
    if length > 8:
        freq[-1, -1, pf:length - pr] += 1.0
        freq[-1, -1, pf] = 0.5                             # the first candidate
        freq[-1, 0, length - 1 - pr] = -0.0                # the last candidate, with a signed zero
    okc, ovc, opos, ofreq = kc.astype(np.float64), vc.astype(np.float64), pos.copy(), freq.copy()
    ovictim = oracle.evict_min(ofreq, okc, ovc, opos, length, pf, pr)

    dkc, dvc, dpos, dfreq = to_dev(kc, dtype), to_dev(vc, dtype), torch.from_numpy(pos).cuda(), torch.from_numpy(freq).cuda()
    dvic = torch.full((B, G), -1, dtype=torch.int32, device="cuda")
    ec.ec_evict_min(dkc, dvc, dpos, dfreq, length, pf, pr, dvic)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(dvic.cpu().numpy(), ovictim)
    m = length - 1
    np.testing.assert_array_equal(to_host(dkc)[:, :, :m], okc[:, :, :m])
    np.testing.assert_array_equal(to_host(dvc)[:, :, :m], ovc[:, :, :m])
    np.testing.assert_array_equal(dpos.cpu().numpy()[:, :, :m], opos[:, :, :m])
    np.testing.assert_array_equal(dfreq.cpu().numpy()[:, :, :m].view(np.int32), ofreq[:, :, :m].view(np.int32))
    # nothing beyond the old end is touched
    np.testing.assert_array_equal(to_host(dkc)[:, :, length:], kc[:, :, length:].astype(np.float64))
    np.testing.assert_array_equal(dfreq.cpu().numpy()[:, :, length:], freq[:, :, length:])


@pytest.mark.parametrize("length", [64, 1025, 1026])      # one wave's worth of masses; either side of one workgroup's
def test_evict_min_of_infinite_masses(length):
    """Masses of +inf are ordinary values: the first candidate among equals, and finite ones before them."""
    kc = torch.arange(length, dtype=torch.float32, device="cuda")[None, None, :, None].expand(1, 1, length, 64).contiguous()
    for finite_at, expect in ((None, 3), (length - 2, length - 2)):
        dkc, dvc = kc.clone(), -kc
        freq = torch.full((1, 1, length), float("inf"), device="cuda")
        if finite_at is not None:
            freq[0, 0, finite_at] = 3e38
        victim = torch.full((1, 1), -1, dtype=torch.int32, device="cuda")
        ec.ec_evict_min(dkc, dvc, None, freq, length, 3, 1, victim)
        torch.cuda.synchronize()
        assert victim.item() == expect
        left = torch.cat([kc[0, 0, :expect], kc[0, 0, expect + 1:]])
        assert torch.equal(dkc[0, 0, :length - 1], left) and torch.equal(dvc[0, 0, :length - 1], -left)
        assert torch.isinf(freq[0, 0, :length - 1]).all()


@pytest.mark.parametrize("bits", [0x7fc00000, 0xffc00000, 0xff800001])
def test_evict_min_of_masses_that_are_not_numbers(bits):
    """NaN of either sign never goes before a number."""
    length, least = 700, 333
    kc = torch.arange(length, dtype=torch.float32, device="cuda")[None, None, :, None].expand(1, 1, length, 64).contiguous()
    mass = np.linspace(1.0, 2.0, length, dtype=np.float32)
    mass[[5, 100, 301, 650]] = np.array([bits], np.uint32).view(np.float32)
    for value in (0.5, np.inf):
        mass[least] = value
        if value == np.inf:   # +inf is the only number left
            mass[np.arange(length) != least] = np.array([bits], np.uint32).view(np.float32)
        freq, victim = torch.from_numpy(mass.copy()[None, None]).cuda(), torch.full((1, 1), -1, dtype=torch.int32, device="cuda")
        ec.ec_evict_min(kc.clone(), -kc, None, freq, length, 3, 1, victim)
        torch.cuda.synchronize()
        assert victim.item() == least


def test_frequency_generation_against_the_oracle():
    """Forty generated tokens under the frequency policy at a fixed budget.  Each step the oracle's own
    counts (rounded to fp32) are what both sides choose the victim from."""
    dtype, B, H, D, n0, steps = "bf16", 2, 4, 128, 120, 40
    cap = n0 + 2
    rng = np.random.default_rng(99)
    kc, vc = _cache(rng, B, H, cap, n0, D, dtype)
    scale = 1.0 / np.sqrt(D)
    pos = np.zeros((B, 1, cap), np.int32); pos[:, :, :n0] = np.arange(n0)
    freq0 = (rng.random((B, 1, cap)) * 0.03).astype(np.float32)   # low enough for cached rows to compete with new ones
    okc, ovc, opos, ofreq = kc.astype(np.float64), vc.astype(np.float64), pos.copy(), freq0.astype(np.float64)
    dkc, dvc, dpos, dfreq = to_dev(kc, dtype), to_dev(vc, dtype), torch.from_numpy(pos).cuda(), torch.from_numpy(freq0).cuda()
    dout = torch.empty((B, H, D), dtype=torch.bfloat16, device="cuda")
    dvic = torch.empty((B, 1), dtype=torch.int32, device="cuda")
    ws = ec.new_workspace(ec.EC_FN_DECODE_SCORE_STEP, B, H, cap, D, ec.EC_BF16)
    N = n0
    victims = []
    for s in range(steps):
        q, kn, vn = (quantize(rng.standard_normal((B, H, D)), dtype) for _ in range(3))
        oout, _ = oracle.decode_score_step(q, kn, vn, okc, ovc, opos, ofreq, N, 1000 + s, scale)
        ec.ec_decode_score_step(to_dev(q, dtype), to_dev(kn, dtype), to_dev(vn, dtype), dkc, dvc, dpos, dfreq, N,
                                1000 + s, scale, dout, ws)
        torch.cuda.synchronize()
        assert_close(to_host(dout), oout, dtype, f"out step {s}")
        assert np.abs(dfreq.cpu().numpy()[:, :, :N + 1] - ofreq[:, :, :N + 1]).max() <= 2e-3
        if ec.ec_evict_index(1000 + s, N + 1, 1, 1, budget_mode=ec.EC_BUDGET_FIXED, fixed_len=n0) >= 0:
            f32 = ofreq.astype(np.float32)
            dfreq.copy_(torch.from_numpy(f32))            # both sides decide on the same fp32 counts
            victims.append(oracle.evict_min(f32, okc, ovc, opos, N + 1, 1, 1))
            ofreq = f32.astype(np.float64)
            ec.ec_evict_min(dkc, dvc, dpos, dfreq, N + 1, 1, 1, dvic)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(dvic.cpu().numpy(), victims[-1])
        else:
            N += 1
    assert len(victims) == steps and N == n0
    np.testing.assert_array_equal(to_host(dkc)[:, :, :N], okc[:, :, :N])
    np.testing.assert_array_equal(dpos.cpu().numpy()[:, :, :N], opos[:, :, :N])
    assert len({int(v[0, 0]) for v in victims}) >= 2       # not always the same row
