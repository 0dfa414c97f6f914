"""Losses of heads whose logits stay in registers and are sorted in runs of 32 (more than 8192 tokens, at most 32768):
lengths at the edges of the register counts and of the runs, one and several shares per head, and clusters of equal
logits around the 17 that a run takes care of, above which a finer bin is put in order by itself or the share is sorted."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


def losses(dev, K, Q, rank, m):
    Hkv, T = K.shape[1:3]
    Hq = Q.shape[1]
    ws = torch.full((l2kv.l2kv_alr_workspace_bytes(1, Hq, T),), 0xA5, dtype=torch.uint8, device=dev)
    runs = []
    for _ in range(2):
        out = [torch.full((1, Hq), float("nan"), dtype=torch.float64, device=dev) for _ in range(3)]
        l2kv.l2kv_alr(Q, K, rank, m, *out, ws)
        runs.append([o.cpu().numpy() for o in out])
    for a, b in zip(*runs):
        assert np.array_equal(a, b, equal_nan=True)                   # same bits whatever the order of arrival
    return runs[0]


# 16, 20, 24 and 32 keys per lane; with 2 heads up to 16 shares of 2048, with 256 one of up to 19452
@pytest.mark.parametrize("T,Hkv,G", [(8193, 1, 2), (16384, 1, 2), (16385, 1, 2), (20480, 1, 2), (20481, 1, 2), (24577, 1, 2), (32767, 1, 2),
                                     (32768, 1, 2), (8224, 32, 8), (16384, 32, 8), (19452, 32, 8), (19453, 32, 8)])
@pytest.mark.parametrize("each", [1, 9, 17, 18, 40])
def test_losses(dev, T, Hkv, G, each):
    rng = np.random.default_rng(T + each)
    rows = (T + each - 1) // each
    K = rng.standard_normal((1, Hkv, rows, 64)) * np.exp(0.5 * rng.standard_normal((1, Hkv, rows, 1)))
    K = torch.from_numpy(K.astype(np.float32)).to(torch.bfloat16)[:, :, torch.from_numpy(rng.permutation(rows * each)[:T] // each)].contiguous()
    Q = torch.from_numpy(rng.standard_normal((1, Hkv * G, 64)).astype(np.float32)).to(torch.bfloat16)
    Kd = K.to(dev)
    norms = torch.empty((1, Hkv, T), device=dev)
    l2kv.l2kv_norms(Kd, norms)
    rank = torch.empty((1, Hkv, T), dtype=torch.int32, device=dev)
    l2kv.l2kv_norm_ranks(norms, rank, torch.empty(l2kv.l2kv_norm_ranks_workspace_bytes(Hkv, T), dtype=torch.uint8, device=dev))
    m = T // 3
    got = losses(dev, Kd, Q.to(dev), rank, m)
    for h in {0, Hkv - 1}:
        Qn, Kn = synth.as_numpy_bits(Q[:, h * G:h * G + 2].contiguous()), synth.as_numpy_bits(K[:, h:h + 1].contiguous())
        want = oracle.alr_heads(Qn, Kn, norms[:, h:h + 1].cpu().numpy(), "bf16", m)
        Y, Lm, Lref = (x[:, h * G:h * G + 2] for x in got)
        # scores are fp32 sums of 64 products and an exp2 of 1-2 ulp, about 1e-6 relative each; losses are sums of them (at
        # most 1), Y weights them with integers up to T
        assert np.abs(Y - want[0]).max() <= 2e-6 * T
        assert np.abs(Lm - want[1]).max() <= 2e-6 and np.abs(Lref - want[2]).max() <= 2e-6


@pytest.mark.parametrize("T", [9000, 32768])
def test_logits_that_are_not_finite(dev, T):
    """A key row that makes a logit of -inf takes no part; one that makes +inf or NaN leaves no number."""
    g = torch.Generator(device=dev)
    g.manual_seed(T)
    K = torch.randn((1, 4, T, 64), generator=g, device=dev)
    Q = torch.randn((1, 4, 64), generator=g, device=dev)
    K[0, 1, 5] = torch.where(Q[0, 1] > 0, -torch.inf, torch.inf)
    K[0, 2, 5] = torch.where(Q[0, 2] > 0, torch.inf, -torch.inf)
    K[0, 3, 5, 7] = torch.nan
    rank = torch.argsort(torch.rand((1, 4, T), generator=g, device=dev), dim=-1).int()
    got = losses(dev, K, Q, rank, T // 2)
    for x in got:
        assert np.isfinite(x[0, :2]).all() and np.isnan(x[0, 2:]).all()
    K[0, 1, 5] *= 0.0
    K[0, 1, 5] = -1e4 * Q[0, 1]                                        # a logit far below all others
    assert all(np.allclose(a[0, 1], b[0, 1], rtol=1e-6, atol=0) for a, b in zip(got, losses(dev, K, Q, rank, T // 2)))


# Groups of equal logits that fill finer bins: up to 17 for a run, 32 for a piece, 64 for two, more for the exact cut.
@pytest.mark.parametrize("T,Hkv,B", [(8193, 2, 1), (16384, 2, 1), (20481, 2, 1), (32768, 2, 1), (12000, 32, 4), (16384, 32, 8), (19452, 32, 8),
                                     (32768, 32, 4)])
@pytest.mark.parametrize("each", [1, 9, 17, 18, 25, 32, 33, 40, 64, 65])
def test_order(dev, T, Hkv, B, each):
    """With the ranks of the scores themselves as the order of discarding, both terms of Y are the same sum of the same
    numbers, and so are both losses: a score out of place shows even where its neighbours are nearly equal."""
    g = torch.Generator(device=dev).manual_seed(T + each)
    rows = (T + each - 1) // each
    K = torch.randn((B, Hkv, rows, 64), generator=g, device=dev) * torch.exp(0.5 * torch.randn((B, Hkv, rows, 1), generator=g, device=dev))
    K = K.bfloat16()[:, :, torch.randperm(rows * each, generator=g, device=dev)[:T] // each].contiguous()
    Q = torch.randn((B, Hkv, 64), generator=g, device=dev).bfloat16()
    rank = torch.zeros((B, Hkv, T), dtype=torch.int32, device=dev)
    ws = torch.empty(l2kv.l2kv_alr_workspace_bytes(B, Hkv, T), dtype=torch.uint8, device=dev)
    Y, Lm, Lref = (torch.empty((B, Hkv), dtype=torch.float64, device=dev) for _ in range(3))
    m = T // 3
    l2kv.l2kv_alr(Q, K, rank, m, Y, Lm, Lref, ws)
    logits = ws[:B * Hkv * T * 4].view(torch.float32).view(B, Hkv, T)          # left at its start
    exact = torch.einsum("bhd,bhtd->bht", Q.cpu().float(), K[:, :, :64].cpu().float()) / 8 * 1.4426950408889634
    assert (logits[:, :, :64].cpu() - exact).abs().max() <= 1e-4               # these are they; 64 products of up to 1e2 in fp32
    rank.scatter_(2, torch.argsort(logits, dim=2, stable=True), torch.arange(T, dtype=torch.int32, device=dev).expand(B, Hkv, T).contiguous())
    l2kv.l2kv_alr(Q, K, rank, m, Y, Lm, Lref, ws)
    # sums in 64 bits of at most T numbers that add up to 1, times at most T: no term takes part in more than 100 additions (32 by a
    # lane, the waves', the shares'), in both terms of Y
    assert Y.abs().max() <= 2 * 128 * 2.0 ** -53 * T
    assert (Lm - Lref).abs().max() <= 2 * 128 * 2.0 ** -53
