"""Decode attention over heads so short that one workgroup takes each, and over a few heads of long rows, whose splits are counted in
64-row blocks: the plan at the edges of both rules, and the result against fp64."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


def run(dtype, D, G, heads, n, splits):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n + G)
    Q = (2 * torch.randn((1, heads * G, D), generator=g, device=dev)).to(dtype)
    K, V = (torch.randn((1, heads, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    O, same, other = (torch.full((1, heads * G, D), float("nan"), device=dev) for _ in range(3))
    l2kv.l2kv_decode_attn(Q, K, V, O, ws)
    binding.l2kv_decode_attn_splits(Q, K, V, same, ws, n_splits=splits)
    binding.l2kv_decode_attn_splits(Q, K, V, other, ws, n_splits=splits // 2 if splits > 1 else 2)
    assert torch.equal(O, same) and not torch.equal(O, other)           # the same plan: the same order of the sums
    q, k, v = Q.cpu().double(), K.cpu().double(), V.cpu().double()
    k, v = (x.repeat_interleave(G, dim=1) for x in (k, v))
    p = torch.softmax((k @ q[..., None])[..., 0] / math.sqrt(D), dim=-1)
    want = (p[..., None] * v).sum(dim=2)
    # fp32 sums of at most (n / 16 rows + the merges) terms of magnitude max |V| < 6 times weights that add up to 1
    assert (O.cpu().double() - want).abs().max() <= (n / 16 + 64) * 2.0 ** -24 * 6


@pytest.mark.parametrize("dtype,D,G,one,more", [(torch.bfloat16, 128, 1, (65, 256), (257,)), (torch.bfloat16, 128, 3, (128, 192), (193,)), (torch.bfloat16, 128, 8, (65, 128), (129,)),
                                                (torch.bfloat16, 64, 2, (129, 512), (513,)), (torch.bfloat16, 64, 3, (384,), (385,)), (torch.bfloat16, 64, 4, (256,), (257,)),
                                                (torch.bfloat16, 256, 3, (65, 128), (129,)), (torch.bfloat16, 256, 4, (), (65,)), (torch.float32, 64, 2, (65, 256), (257,)),
                                                (torch.float32, 128, 2, (65, 128), (129,)), (torch.float32, 128, 4, (), (65, 128))])
def test_one_workgroup(dtype, D, G, one, more):
    for n in one:
        run(dtype, D, G, 5, n, 1)
    for n in more:
        run(dtype, D, G, 5, n, min(8, l2kv.l2kv_decode_max_splits(n)))


@pytest.mark.parametrize("dtype,D,G,heads,n,splits", [(torch.float32, 128, 1, 1, 800, 13), (torch.float32, 128, 2, 3, 1886, 30), (torch.float32, 128, 1, 1, 9322, 49), (torch.bfloat16, 256, 3, 3, 4121, 33),
                                                      (torch.float32, 128, 1, 4, 768, 8), (torch.bfloat16, 256, 2, 1, 53342, 167), (torch.bfloat16, 256, 1, 4, 8192, 43), (torch.bfloat16, 256, 1, 4, 8193, 30)])
def test_few_heads_of_long_rows(dtype, D, G, heads, n, splits):
    run(dtype, D, G, heads, n, splits)
