"""Compression with rows of V requested before the search: shares of tokens of one head (selection with copy) and of a whole
head with its norms (one launch), at the edges of the shares and of the rules that choose them, against the three
separate calls."""
import pytest
import torch

import paper_2406_11430_amd as l2kv
from test_gpu_compress_short import separate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


ROWS = [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256), (torch.float32, 64), (torch.float32, 128)]
# one launch up to 128 KB a head: shares of 64 tokens, of as many as one workgroup on a compute unit leaves, of the most a
# workgroup holds; heads beyond the number of compute dies, one more head than shares fit
SHORT = [(1, 63), (3, 64), (7, 65), (8, 127), (9, 128), (17, 256), (33, 200), (64, 255), (128, 257), (129, 256), (256, 128), (256, 17),
         (2, 512), (5, 511), (2, 513), (16, 1024)]
# two launches: shares of 64 tokens, of the most a workgroup holds and of one too many, last shares of a few tokens
AHEAD = [(1, 1025), (2, 3001), (8, 2049), (31, 4096), (33, 4096), (60, 1111), (120, 1030), (8, 4097), (7, 8191), (9, 8192), (128, 1040)]


@pytest.mark.parametrize("dtype,D", ROWS)
@pytest.mark.parametrize("heads,T", SHORT + AHEAD)
@pytest.mark.parametrize("kept", ["third", "below_third", "all"])
def test_tokens_of_a_share(dev, dtype, D, heads, T, kept):
    k = {"third": (T + 2) // 3, "below_third": max(1, (T + 2) // 3 - 1), "all": T}[kept]
    g = torch.Generator(device=dev).manual_seed(31 * T + heads)
    K = torch.randn((heads, T, D), generator=g, device=dev)
    V = torch.randn((heads, T, D), generator=g, device=dev).to(dtype)
    # kept tokens of the even heads all in one stretch, so that some shares keep every row and others none; ties across it
    K[::2, T // 4:T // 4 + k] *= 0.01
    K[::2, T // 4:T // 4 + k:3] = K[::2, T // 4:T // 4 + 1].clone()
    K[1::2, ::5] = 0.0
    K = K.to(dtype)
    norms = torch.full((heads, T), -1.0, device=dev)
    idx = torch.full((heads, k), -1, dtype=torch.int32, device=dev)
    Kc, Vc = (torch.zeros((heads, k, D), dtype=dtype, device=dev) for _ in range(2))
    ws = torch.zeros(256, dtype=torch.uint8, device=dev)
    ratio = next(r for r in (k / T, (k - 0.5) / T) if l2kv.l2kv_keep_count(T, r) == k)
    l2kv.l2kv_compress(K, V, ratio, norms, idx, Kc, Vc, ws)
    for got, want in zip((norms, idx, Kc, Vc), separate(K, V, k)):
        assert torch.equal(got, want)


# K just within and just outside the sizes of which the norm pass leaves everything in the caches, little kept
@pytest.mark.parametrize("heads", [40, 41, 96, 97])
def test_little_kept_of_a_cached_k(dev, heads):
    g = torch.Generator(device=dev).manual_seed(heads)
    K, V = (torch.randn((heads, 4096, 128), generator=g, device=dev).bfloat16() for _ in range(2))
    k = l2kv.l2kv_keep_count(4096, 0.1)
    norms, idx = torch.empty((heads, 4096), device=dev), torch.empty((heads, k), dtype=torch.int32, device=dev)
    Kc, Vc = (torch.empty((heads, k, 128), dtype=K.dtype, device=dev) for _ in range(2))
    l2kv.l2kv_compress(K, V, 0.1, norms, idx, Kc, Vc, torch.zeros(256, dtype=torch.uint8, device=dev))
    for got, want in zip((norms, idx, Kc, Vc), separate(K, V, k)):
        assert torch.equal(got, want)
