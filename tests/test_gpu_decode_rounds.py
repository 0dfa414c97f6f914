"""Decode attention over so many heads that one workgroup each would leave the last round of compute units half idle: the split count on
either side of the lines, the result against fp64 and the scratch memory of the entry point without a workspace."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


def operands(dtype, D, G, heads, n):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n + heads)
    Q = (2 * torch.randn((1, heads * G, D), generator=g, device=dev)).to(dtype)
    K, V = (torch.randn((1, heads, n, D), generator=g, device=dev, dtype=torch.float32).to(dtype) for _ in range(2))
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    return Q, K, V, ws


@pytest.mark.parametrize("dtype,D,G,heads,n,splits", [
    (torch.bfloat16, 128, 1, 85, 400, 3), (torch.bfloat16, 128, 1, 86, 400, 2), (torch.bfloat16, 128, 4, 56, 400, 4), (torch.bfloat16, 128, 4, 58, 400, 3), (torch.float32, 128, 2, 80, 300, 3),
    (torch.bfloat16, 64, 8, 163, 4096, 3), (torch.bfloat16, 64, 8, 163, 4095, 1), (torch.bfloat16, 64, 8, 164, 4096, 1), (torch.bfloat16, 64, 5, 129, 4100, 3),
    (torch.bfloat16, 128, 1, 146, 8192, 3), (torch.bfloat16, 128, 1, 147, 8192, 1), (torch.bfloat16, 128, 3, 146, 8191, 1), (torch.float32, 128, 7, 130, 2048, 3),
    (torch.bfloat16, 64, 1, 257, 3072, 3), (torch.bfloat16, 64, 1, 257, 3071, 1), (torch.bfloat16, 64, 4, 341, 3072, 3), (torch.bfloat16, 64, 1, 342, 3072, 1),
    (torch.bfloat16, 64, 4, 342, 3072, 2), (torch.bfloat16, 64, 4, 384, 3072, 2), (torch.bfloat16, 64, 4, 385, 3072, 1), (torch.float32, 128, 6, 260, 1535, 1), (torch.float32, 128, 6, 260, 1536, 3),
    (torch.bfloat16, 64, 2, 513, 5120, 3), (torch.bfloat16, 64, 2, 597, 5120, 3), (torch.bfloat16, 64, 2, 598, 5120, 1), (torch.bfloat16, 64, 2, 513, 5119, 1),
    (torch.bfloat16, 64, 6, 97, 8192, 5), (torch.bfloat16, 64, 6, 98, 8192, 2), (torch.bfloat16, 64, 6, 97, 8191, 2)])
def test_splits(dtype, D, G, heads, n, splits):
    Q, K, V, ws = operands(dtype, D, G, heads, n)
    O, same, other = (torch.full((1, heads * G, D), float("nan"), device=Q.device) for _ in range(3))
    l2kv.l2kv_decode_attn(Q, K, V, O, ws)
    binding.l2kv_decode_attn_splits(Q, K, V, same, ws, n_splits=splits)
    binding.l2kv_decode_attn_splits(Q, K, V, other, ws, n_splits=splits + 1)
    assert torch.equal(O, same) and not torch.equal(O, other)           # the same plan: the same order of the sums
    for head in (0, heads // 2, heads - 1):
        q, k, v = Q[0, head * G:(head + 1) * G].cpu().double(), K[0, head].cpu().double(), V[0, head].cpu().double()
        want = torch.softmax(q @ k.T / math.sqrt(D), dim=-1) @ v
        # fp32 sums of at most (n / 16 rows + the merges) terms of magnitude max |V| < 6 times weights that add up to 1
        assert (O[0, head * G:(head + 1) * G].cpu().double() - want).abs().max() <= (n / 16 + 64) * 2.0 ** -24 * 6


@pytest.mark.parametrize("G,splits", [(4, 3), (8, 1)])
def test_without_a_workspace(G, splits):
    """Three partial results of 341 heads with 8 query heads find no room in the static scratch memory, which one does not need."""
    Q, K, V, ws = operands(torch.bfloat16, 128, G, 341, 1536)
    O, want = (torch.full((1, 341 * G, 128), float("nan"), device=Q.device) for _ in range(2))
    binding.l2kv_decode_attn_static(Q, K, V, O)
    binding.l2kv_decode_attn_splits(Q, K, V, want, ws, n_splits=splits)
    assert torch.equal(O, want)


@pytest.mark.parametrize("dtype,D,G,heads,n", [(torch.bfloat16, 128, 8, 544, 4096), (torch.bfloat16, 256, 4, 513, 1500), (torch.float32, 128, 5, 530, 2600), (torch.bfloat16, 128, 8, 331, 2048),
                                               (torch.float32, 128, 5, 529, 2600), (torch.bfloat16, 128, 8, 330, 2048)])
def test_same_without_a_workspace(dtype, D, G, heads, n):
    Q, K, V, ws = operands(dtype, D, G, heads, n)
    O, want = (torch.full((1, heads * G, D), float("nan"), device=Q.device) for _ in range(2))
    binding.l2kv_decode_attn_static(Q, K, V, O)
    l2kv.l2kv_decode_attn(Q, K, V, want, ws)
    assert torch.equal(O, want)
