"""fp32 scoring: column masses of keys whose probabilities are subnormal numbers (the exponential instruction alone gives
zero there), beside ordinary ones, at odd and even numbers of tiles."""
import pytest
import torch

from paper_2407_18121_amd import binding as ec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,T", [(1, 33), (2, 100), (40, 200), (40, 520)])
def test_subnormal_probabilities(H, T, D):
    g = torch.Generator().manual_seed(T + D)
    q, k, v = (torch.zeros(1, H, T, D) for _ in range(3))
    q[..., 0] = 1.0
    k[..., 0] = torch.randint(0, 3, (1, H, T), generator=g).float()
    k[:, :, 0, 0] = 95.0                 # takes all the mass
    k[:, :, 1::3, 0] = 1.5               # exp(-93.5) = 2.5e-41
    k[:, :, 2::7, 0] = 0.0               # exp(-95) = 5.5e-42
    v[..., 0] = 1.0
    score = torch.zeros(1, H, T, device="cuda")
    out = torch.zeros(1, H, T, D, device="cuda")
    ws = ec.new_workspace(ec.EC_FN_PREFILL_SCORE, 1, H, T, D, ec.EC_F32)
    ec.ec_prefill_score(q.cuda(), k.cuda(), v.cuda(), out, None, score, 1.0, ws)
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous())
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool).triu(1), -torch.inf)
    want = torch.softmax(s, -1).sum(-2)
    # a probability is off by the rounding of its exponent, about 95 / ln 2 * 2^-24 twice, and by half of the smallest subnormal
    # number (1.4e-45) for each of up to T summands
    assert ((score.cpu().double() - want).abs() <= 4e-5 * want + 0.7e-45 * T).all()
    assert (score.cpu()[:, :, 1:] > 0).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,T", [(1, 33), (2, 100), (40, 200), (40, 520)])
@pytest.mark.parametrize("at", ["first", "middle"])
def test_output_of_subnormal_probabilities(H, T, D, at):
    """The key that takes all the mass has no V; all others, before and behind it, have V of 1e34 and more."""
    g = torch.Generator().manual_seed(T + D)
    n = 0 if at == "first" else T // 2
    q, k = (torch.zeros(1, H, T, D) for _ in range(2))
    q[..., 0] = 1.0
    k[..., 0] = -88.5 - 2 * torch.rand(1, H, T, generator=g)     # 2^-127.7 to 2^-130.6
    v = 1e34 * (1 + torch.rand(1, H, T, D, generator=g))
    k[:, :, n, 0], v[:, :, n] = 0.0, 0.0
    score, out = torch.zeros(1, H, T, device="cuda"), torch.zeros(1, H, T, D, device="cuda")
    ws = ec.new_workspace(ec.EC_FN_PREFILL_SCORE, 1, H, T, D, ec.EC_F32)
    ec.ec_prefill_score(q.cuda(), k.cuda(), v.cuda(), out, None, score, 1.0, ws)
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous())
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool).triu(1), -torch.inf)
    want = torch.matmul(torch.softmax(s, -1), v.double())
    # scores of up to 131 in base-2 units, three roundings of 2^-24 each, are exponents: 131 * 3 * 2^-24 * ln 2 < 2^-15
    torch.testing.assert_close(out.cpu().double(), want, rtol=2 ** -15, atol=0)
