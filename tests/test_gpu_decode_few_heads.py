"""Decode attention over one to four heads: the split count that the steps of the longest split and the merge ask for, on either side of the
lines of that rule, and the result against fp64."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,G,heads,n,splits", [
    (torch.bfloat16, 128, 1, 1, 16000, 63), (torch.bfloat16, 128, 4, 2, 4096, 32), (torch.bfloat16, 128, 4, 3, 4096, 21), (torch.bfloat16, 128, 8, 2, 4096, 32),
    (torch.float32, 128, 8, 1, 4096, 32), (torch.float32, 128, 8, 4, 4096, 32), (torch.float32, 128, 8, 5, 4096, 21), (torch.float32, 64, 4, 1, 3072, 24),
    (torch.float32, 64, 4, 1, 3071, 18), (torch.bfloat16, 128, 1, 1, 32768, 64), (torch.bfloat16, 128, 1, 1, 32769, 61), (torch.bfloat16, 128, 5, 1, 65536, 128),
    (torch.bfloat16, 64, 2, 1, 16000, 43)])
def test_splits(dtype, D, G, heads, n, splits):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n + G)
    Q = (2 * torch.randn((1, heads * G, D), generator=g, device=dev)).to(dtype)
    K, V = (torch.randn((1, heads, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    O, same, other = (torch.full((1, heads * G, D), float("nan"), device=dev) for _ in range(3))
    l2kv.l2kv_decode_attn(Q, K, V, O, ws)
    binding.l2kv_decode_attn_splits(Q, K, V, same, ws, n_splits=splits)
    binding.l2kv_decode_attn_splits(Q, K, V, other, ws, n_splits=splits // 2)
    assert torch.equal(O, same) and not torch.equal(O, other)           # the same plan: the same order of the sums
    q, k, v = Q.cpu().double(), K.cpu().double(), V.cpu().double()
    k, v = (x.repeat_interleave(G, dim=1) for x in (k, v))
    p = torch.softmax((k @ q[..., None])[..., 0] / math.sqrt(D), dim=-1)
    want = (p[..., None] * v).sum(dim=2)
    # fp32 sums of at most (n / 16 rows + the merges) terms of magnitude max |V| < 6 times weights that add up to 1
    assert (O.cpu().double() - want).abs().max() <= (n / 16 + 64) * 2.0 ** -24 * 6
