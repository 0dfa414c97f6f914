"""Ranking of heads whose keys the bins do not separate: clusters of equal norms and logits below and above
what a bin may hold, one outlier that stretches the bins of a long head, long heads in many shares, and
the counting passes of many long heads.  The ranks are whole numbers and must match the order of (norm bits,
position) exactly."""
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


def levels(rng, T, each):
    """About `each` equal keys per value, values over a few octaves."""
    return np.exp2(rng.integers(0, max(1, T // each), T) / 8.0 % 16.0).astype(np.float32)


def key_sets(rng, T):
    log = np.exp(rng.standard_normal(T)).astype(np.float32) * 128
    zero = log.copy()
    zero[T // 3] = 0.0                                                # one padded row
    zeros = log.copy()
    zeros[rng.permutation(T)[:T // 3]] = 0.0
    two = np.where(rng.random(T) < 0.5, np.float32(1.0), np.float32(np.nextafter(np.float32(1.0), 2, dtype=np.float32)))
    wide = rng.integers(0, 2 ** 32, T, dtype=np.uint64).astype(np.uint32)      # any bit pattern, the largest among them
    wide[rng.permutation(T)[:T // 4]] = 0xFFFFFFFF
    token = rng.zipf(1.2, T) % 5000                                   # repeated tokens: a norm per token
    return np.stack([log, zero, zeros, levels(rng, T, 100), levels(rng, T, 900), levels(rng, T, 1100), two.astype(np.float32),
                     wide.view(np.float32), np.exp(np.random.default_rng(1).standard_normal(5000))[token].astype(np.float32)])


def ranks(dev, norms):
    d = torch.from_numpy(norms).to(dev)
    rank = torch.full(norms.shape, -1, dtype=torch.int32, device=dev)
    ws = torch.full((l2kv.l2kv_norm_ranks_workspace_bytes(*norms.shape),), 0xA5, dtype=torch.uint8, device=dev)
    l2kv.l2kv_norm_ranks(d, rank, ws)
    return rank.cpu().numpy()


def expected(norms):
    want = np.empty(norms.shape, np.int32)
    for h in range(len(norms)):
        order = oracle.drop_order(norms[h])
        want[h, order] = np.arange(norms.shape[1], dtype=np.int32)
    return want


# 8192 / 32768: where the keys of the bins leave the registers; 9212 / 18424: one share more; 131072: 15 shares
@pytest.mark.parametrize("T", [2, 63, 1025, 4096, 8191, 8193, 9213, 18425, 32768, 32769, 131072])
def test_norm_ranks(dev, T):
    norms = key_sets(np.random.default_rng(T), T)
    assert np.array_equal(ranks(dev, norms), expected(norms))


# one workgroup per head up to 1024 elements, and up to 2048 from 512 heads on
@pytest.mark.parametrize("T", [1, 64, 65, 1000, 1024, 1025, 2000, 2048, 2049])
@pytest.mark.parametrize("heads", [9, 513])
def test_short_heads(dev, heads, T):
    one = key_sets(np.random.default_rng(T), T)
    norms = np.ascontiguousarray(one[np.arange(heads) % len(one)])
    assert np.array_equal(ranks(dev, norms), expected(one)[np.arange(heads) % len(one)])


# 65 shares of a head of 600k, all heads by the passes (64 x 66 shares would be too many), 4M elements in a bin's range
@pytest.mark.parametrize("heads,T", [(1, 599999), (64, 600001), (1, 4194305)])
def test_long_heads(dev, heads, T):
    rng = np.random.default_rng(T)
    norms = (np.exp(rng.standard_normal((heads, T), np.float32)) * 128).astype(np.float32)
    norms[0, ::5] = 7.0
    got = ranks(dev, norms)
    for h in {0, heads - 1}:
        assert np.array_equal(got[h], expected(norms[h:h + 1])[0])


# rows repeated a few hundred times: clusters of equal logits below (300, 900) and above (1100) what a bin may hold
@pytest.mark.parametrize("T,Hkv,G", [(1, 1, 1), (700, 2, 4), (1024, 1, 3), (1025, 1, 2), (1500, 64, 8), (2049, 1, 1), (4096, 2, 4),
                                     (10241, 1, 2), (19453, 2, 4), (45000, 1, 2)])
@pytest.mark.parametrize("each", [100, 300, 900, 1100])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_alr(dev, T, Hkv, G, each, dtype):
    rng = np.random.default_rng(T + each)
    rows = max(2, T // each)
    K = (rng.standard_normal((1, Hkv, rows, 128)) * np.exp(0.5 * rng.standard_normal((1, Hkv, rows, 1)))).astype(np.float32)
    K = np.ascontiguousarray(K[:, :, rng.integers(0, rows, T)])
    K, Q = (torch.from_numpy(x.astype(np.float32)).to(dtype) for x in (K, rng.standard_normal((1, Hkv * G, 128))))
    Kd, Qd = K.to(dev), Q.to(dev)
    norms = torch.empty((1, Hkv, T), device=dev)
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
        assert np.array_equal(a, b)                                   # same bits whatever the order of arrival
    Qn, Kn = (synth.as_numpy_bits(x) if dtype == torch.bfloat16 else x.numpy() for x in (Q, K))
    want = oracle.alr_heads(Qn, Kn, norms.cpu().numpy(), "bf16" if dtype == torch.bfloat16 else "f32", m)
    # scores are fp32 sums of 128 products and an exp2 of 1-2 ulp, about 1e-6 relative each; losses are sums of them
    # (at most 1), Y weights them with integers up to T
    assert np.abs(runs[0][0] - want[0]).max() <= 2e-6 * T
    assert np.abs(runs[0][1] - want[1]).max() <= 2e-6 and np.abs(runs[0][2] - want[2]).max() <= 2e-6


def seconds(f):
    for _ in range(3):
        f()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("heads,T,each", [(128, 8192, 100), (128, 8192, 300), (128, 8192, 900), (128, 8192, 3000), (1024, 900, 200)])
def test_clusters_do_not_cost_many_times_distinct_keys(dev, heads, T, each):
    """The comparisons inside a bin grow with the square of its equal keys: 128 heads of 8192 took 34 times as long
    at 900 equal norms per value.  A sort of the share instead takes a few times as long."""
    rng = np.random.default_rng(each)
    sets = [(np.exp(rng.standard_normal((heads, T))) * 128).astype(np.float32), np.stack([levels(rng, T, each) for _ in range(heads)])]
    rank = torch.empty((heads, T), dtype=torch.int32, device=dev)
    ws = torch.empty(l2kv.l2kv_norm_ranks_workspace_bytes(heads, T), dtype=torch.uint8, device=dev)
    took = []
    for x in sets:
        d = torch.from_numpy(x).to(dev)
        took.append(seconds(lambda: l2kv.l2kv_norm_ranks(d, rank, ws)))
    assert took[1] <= 6 * took[0], took
