"""Short heads: the one-launch compression and the fused selection and compaction against the three
separate calls, and the threshold search on key sets that fill its bins unevenly."""
import numpy as np
import pytest
import torch

import paper_2406_11430_amd as l2kv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


def separate(K, V, k):
    n, T, D = K.shape
    norms = torch.empty((n, T), device=K.device)
    idx = torch.empty((n, k), dtype=torch.int32, device=K.device)
    Kc = torch.empty((n, k, D), dtype=K.dtype, device=K.device)
    Vc = torch.empty_like(Kc)
    l2kv.l2kv_norms(K, norms)
    l2kv.l2kv_select_k(norms, k, l2kv.L2KV_KEEP_LOWEST, idx, None,
                       torch.empty(l2kv.l2kv_select_workspace_bytes(n, T), dtype=torch.uint8, device=K.device))
    l2kv.l2kv_compact(K, V, idx, Kc, Vc)
    return norms, idx, Kc, Vc


# up to 1024 tokens: one launch (while a head is at most 128 KB); up to 8192: norms, then selection with compaction; beyond: three
@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256),
                                     (torch.float32, 64), (torch.float32, 128)])
@pytest.mark.parametrize("heads,T,ratio", [(1, 1, 1.0), (3, 2, 0.5), (1, 127, 0.3), (2, 1023, 0.51), (5, 1024, 1.0), (40, 1024, 0.01),
                                           (9, 1025, 0.5), (2, 2049, 0.9), (3, 4097, 0.1), (2, 8192, 1.0), (256, 300, 0.7),
                                           (257, 300, 0.7), (2, 8193, 0.5), (200, 130, 0.5), (171, 1100, 0.9), (128, 4097, 0.1),
                                           (129, 4097, 0.1), (3, 8192, 0.9), (127, 4200, 0.05)])
def test_compress_equals_the_three_calls(dev, dtype, D, heads, T, ratio):
    g = torch.Generator(device=dev).manual_seed(T + heads)
    K = torch.randn((heads, T, D), generator=g, device=dev) * torch.exp(0.5 * torch.randn((heads, T, 1), generator=g, device=dev))
    K[:, ::7] = K[:, :1].clone()                                               # ties
    K, V = K.to(dtype), torch.randn((heads, T, D), generator=g, device=dev).to(dtype)
    k = l2kv.l2kv_keep_count(T, ratio)
    norms = torch.full((heads, T), -1.0, device=dev)
    idx = torch.full((heads, k), -1, dtype=torch.int32, device=dev)
    Kc, Vc = (torch.zeros((heads, k, D), dtype=dtype, device=dev) for _ in range(2))
    ws = torch.full((l2kv.l2kv_select_workspace_bytes(heads, T),), 0xA5, dtype=torch.uint8, device=dev)
    l2kv.l2kv_compress(K, V, ratio, norms, idx, Kc, Vc, ws)
    for got, want in zip((norms, idx, Kc, Vc), separate(K, V, k)):
        assert torch.equal(got, want)


# fp32 heads on either side of the sizes and numbers that take one launch
@pytest.mark.parametrize("D,T", [(64, 512), (64, 513), (64, 768), (64, 769), (128, 256), (128, 257), (128, 384), (128, 385)])
@pytest.mark.parametrize("heads", [1, 3, 4, 9, 64, 86, 256])
def test_lines_of_fp32(dev, D, T, heads):
    g = torch.Generator(device=dev).manual_seed(T + heads)
    K, V = (torch.randn((heads, T, D), generator=g, device=dev) for _ in range(2))
    for ratio in (0.07, 0.5, 1.0):
        k = l2kv.l2kv_keep_count(T, ratio)
        out = [torch.full((heads, T), -1.0, device=dev), torch.full((heads, k), -1, dtype=torch.int32, device=dev),
               torch.zeros((heads, k, D), device=dev), torch.zeros((heads, k, D), device=dev)]
        l2kv.l2kv_compress(K, V, ratio, *out, torch.zeros(256, dtype=torch.uint8, device=dev))
        assert all(torch.equal(got, want) for got, want in zip(out, separate(K, V, k)))


def key_sets(rng, T):
    log = (np.exp(rng.standard_normal(T)) * 128).astype(np.float32)
    outliers = log.copy()
    outliers[rng.integers(0, T, 2)] = [0.0, np.inf]                    # stretch the bins over every octave
    zeros = log.copy()
    zeros[rng.permutation(T)[:T // 2]] = 0.0
    few = rng.integers(0, 3, T).astype(np.float32)
    narrow = (np.float32(1.0).view(np.uint32) + rng.integers(0, 300, T).astype(np.uint32)).view(np.float32)
    dense = (np.float32(1.0).view(np.uint32) + rng.integers(0, 1 << 20, T).astype(np.uint32)).view(np.float32)
    dense[0] = np.float32(1e30)                                         # everything else in a few bins: divided again
    largest = np.full(T, np.float32(np.nan))
    largest.view(np.uint32)[:] = 0xFFFFFFFF                             # the pattern of the padding
    return np.stack([log, outliers, zeros, few, narrow, dense, np.full(T, 2.5, np.float32), largest])


@pytest.mark.parametrize("T", [1, 64, 1000, 1024, 2047, 4096, 5000, 16384, 32767, 32768, 32769])
def test_search(dev, T):
    norms = key_sets(np.random.default_rng(T), T)
    bits = norms.view(np.uint32)
    d = torch.from_numpy(norms).to(dev)
    ws = torch.empty(l2kv.l2kv_select_workspace_bytes(len(norms), T), dtype=torch.uint8, device=dev)
    for mode, order in ((l2kv.L2KV_KEEP_LOWEST, bits), (l2kv.L2KV_KEEP_HIGHEST, ~bits)):
        by_key = np.argsort(order, axis=-1, kind="stable")
        for k in sorted({1, (T + 2) // 3, T // 2 + 1 if T > 1 else 1, T}):
            idx = torch.full((len(norms), k), -1, dtype=torch.int32, device=dev)
            l2kv.l2kv_select_k(d, k, mode, idx, None, ws)
            assert np.array_equal(idx.cpu().numpy(), np.sort(by_key[:, :k], axis=-1)), (T, mode, k)
