"""Ranking by value ranges in the attention-loss analysis: head lengths around the switches between
launch shapes (keys in registers or re-read, one or several shares per head), key sets that fill
the bins unevenly, and the exact cut and sort that take over where a bin is too full."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import synth

pytestmark = pytest.mark.gpu

# scores are fp32 sums of 128 products and an exp2 of 1-2 ulp, about 1e-6 relative each; losses
# are sums of them (at most 1), Y weights them with integers up to T
LOSS_BAR = 2e-6
Y_BAR_PER_TOKEN = 2e-6


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


def key_sets(rng, T):
    log = np.exp(rng.standard_normal(T)).astype(np.float32) * 128
    outliers = log.copy()
    outliers[rng.integers(0, T, 3)] = [0.0, np.inf, 1e-38]          # stretch the bins over every octave
    tied = log.copy()
    tied[rng.permutation(T)[:min(1000, T)]] = np.float32(128)        # just below what a bin may hold
    crowded = log.copy()
    crowded[rng.permutation(T)[:max(1, T // 2)]] = 0.0                # far more than that in long heads
    few = rng.integers(0, 5, T).astype(np.float32)
    equal = np.full(T, 2.5, np.float32)
    narrow = (np.float32(1.0).view(np.uint32) + rng.integers(0, 3 * T, T).astype(np.uint32)).view(np.float32)
    rising = np.sort(log)
    return np.stack([log, outliers, tied, crowded, few, equal, narrow, rising])


# 8192 / 32768: keys in registers; 9212: one share to two (lists of keys and positions)
@pytest.mark.parametrize("T", [2, 1023, 2049, 8191, 8192, 8193, 9212, 9213, 32767, 32768, 32769, 50001])
@pytest.mark.parametrize("heads", [8, 5])
def test_norm_ranks(dev, T, heads):
    norms = key_sets(np.random.default_rng(T), T)[:heads] if heads < 8 else key_sets(np.random.default_rng(T), T)
    d = torch.from_numpy(norms).to(dev)
    rank = torch.full(norms.shape, -1, dtype=torch.int32, device=dev)
    ws = torch.empty(l2kv.l2kv_norm_ranks_workspace_bytes(heads, T), dtype=torch.uint8, device=dev)
    l2kv.l2kv_norm_ranks(d, rank, ws)
    got = rank.cpu().numpy()
    for h in range(heads):
        order = oracle.drop_order(norms[h])
        want = np.empty(T, np.int32)
        want[order] = np.arange(T, dtype=np.int32)
        assert np.array_equal(got[h], want), (T, h)


# 19452: one share to two (list of logits); 2049 / 4100 with one query head: shares that fill the chip
@pytest.mark.parametrize("T,Hkv,G", [(2049, 1, 1), (4100, 1, 1), (19452, 2, 4), (19453, 2, 4), (32769, 1, 3), (45000, 1, 2)])
@pytest.mark.parametrize("rows", ["normal", "half zero", "one large", "zero query"])
def test_alr(dev, T, Hkv, G, rows):
    rng = np.random.default_rng(T)
    K = (rng.standard_normal((1, Hkv, T, 128)) * np.exp(0.5 * rng.standard_normal((1, Hkv, T, 1)))).astype(np.float32)
    Q = rng.standard_normal((1, Hkv * G, 128)).astype(np.float32)
    if rows == "half zero":
        K[:, :, rng.permutation(T)[:T // 2]] = 0.0                     # half of the logits equal: cut and sorted
    if rows == "one large":
        K[:, :, 7] *= 30.0                                             # stretches the bins
    if rows == "zero query":
        Q[:] = 0.0
    K, Q = (torch.from_numpy(x).to(torch.bfloat16) for x in (K, Q))
    Kd, Qd = K.to(dev), Q.to(dev)
    norms = torch.empty((1, Hkv, T), dtype=torch.float32, device=dev)
    l2kv.l2kv_norms(Kd, norms)
    rank = torch.empty((1, Hkv, T), dtype=torch.int32, device=dev)
    l2kv.l2kv_norm_ranks(norms, rank, torch.empty(l2kv.l2kv_norm_ranks_workspace_bytes(Hkv, T), dtype=torch.uint8, device=dev))
    m = T // 3
    ws = torch.full((l2kv.l2kv_alr_workspace_bytes(1, Hkv * G, T),), 0xA5, dtype=torch.uint8, device=dev)
    runs = []
    for _ in range(2):
        out = [torch.full((1, Hkv * G), float("nan"), dtype=torch.float64, device=dev) for _ in range(3)]
        l2kv.l2kv_alr(Qd, Kd, rank, m, *out, ws)
        runs.append([o.cpu().numpy() for o in out])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)                                    # same bits whatever the order of arrival
    Y, Lm, Lref = runs[0]
    wY, wLm, wLref = oracle.alr_heads(synth.as_numpy_bits(Q), synth.as_numpy_bits(K), norms.cpu().numpy(), "bf16", m)
    assert np.abs(Y - wY).max() <= Y_BAR_PER_TOKEN * T
    assert np.abs(Lm - wLm).max() <= LOSS_BAR and np.abs(Lref - wLref).max() <= LOSS_BAR
