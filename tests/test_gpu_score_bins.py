"""Order of logits in bins around their mean (heads of 8193 to 32768 tokens): logits far from zero, a few far out on one or both sides, and
bins with more elements than a run takes, up to and beyond what a wave, four waves and the list take care of."""
import numpy as np
import pytest
import torch

import paper_2406_11430_amd as l2kv

pytestmark = pytest.mark.gpu


def rows(kind, n, g):
    x = torch.randn((n,), generator=g, device="cuda:0")
    if kind == "shifted":
        return x * 0.01 - 300.0
    if kind == "one far":
        x[3] = 500.0
    if kind == "two far":
        x[3], x[4] = 3000.0, -1e5
    if kind == "one side":
        x = torch.exp(2.0 * x)
    if kind == "one far below":
        x[3] = -500.0
    if kind == "two far below":
        x[3], x[4] = -3000.0, -1e5
    if kind == "one side below":
        x = -torch.exp(2.0 * x)
    if kind == "narrow":                                               # 17 bits of mantissa left
        x = 1.0 + 1e-2 * x
    return x


# equal logits each: one wave up to 64 and 128, four waves beyond, the exact cut beyond 512
@pytest.mark.parametrize("each", [1, 19, 64, 65, 128, 129, 260, 511, 513])
# (far above, nearly all scores are zero in 32 bits and only their sums are tested; far below, the others keep their scores)
@pytest.mark.parametrize("kind", ["normal", "shifted", "one far", "two far", "one side", "narrow", "one far below", "two far below", "one side below"])
@pytest.mark.parametrize("T,heads", [(8193, 1), (16384, 40), (20479, 256), (32768, 3)])
def test_order(T, heads, kind, each):
    """Keys of one element that is not zero make the logits what they should be.  With the ranks of the logits themselves as the order of discarding, both terms
    of Y are the same sum of the same numbers, and so are both losses: sums in 64 bits of numbers that add up to 1, times at most T, no
    term in more than 100 additions, in both terms of Y.  A logit out of place shows even where its neighbours are nearly equal."""
    g = torch.Generator(device="cuda:0").manual_seed(T + each)
    n = (T + each - 1) // each
    value = rows(kind, n, g)
    K = torch.zeros((1, heads, T, 64), device="cuda:0")
    for h in range(heads):
        K[0, h, :, 5] = value[torch.randperm(n * each, generator=g, device="cuda:0")[:T] // each]
    Q = torch.zeros((1, heads, 64), device="cuda:0")
    Q[..., 5] = 8.0                                                    # the scale is 1 / 8
    logits = K[..., 5]
    counts = torch.exp(logits - logits.amax(dim=2, keepdim=True)) > 0
    assert kind in ("one far", "two far", "one side") or counts.float().mean() > 0.75           # two of 16 values at most are not
    rank = torch.empty((1, heads, T), dtype=torch.int32, device="cuda:0")
    rank.scatter_(2, torch.argsort(logits, dim=2, stable=True), torch.arange(T, dtype=torch.int32, device="cuda:0").expand(1, heads, T).contiguous())
    ws = torch.full((l2kv.l2kv_alr_workspace_bytes(1, heads, T),), 0xA5, dtype=torch.uint8, device="cuda:0")
    Y, Lm, Lref = (torch.empty((1, heads), dtype=torch.float64, device="cuda:0") for _ in range(3))
    m = T // 3
    l2kv.l2kv_alr(Q, K, rank, m, Y, Lm, Lref, ws)
    assert Y.abs().max() <= 2 * 128 * 2.0 ** -53 * T
    assert (Lm - Lref).abs().max() <= 2 * 128 * 2.0 ** -53
    want = torch.sort(torch.softmax(logits.double(), dim=-1), dim=-1).values[..., :m].sum(-1)
    # an fp32 logit of 500 is exact to 3e-5 after the factor log2(e); of those whose scores are not zero
    size = float(torch.where(counts, logits.abs(), 0.0).max())
    assert np.allclose(Lref.cpu().numpy(), want.cpu().numpy(), rtol=2e-6 + 6e-8 * size * 4, atol=1e-300)
