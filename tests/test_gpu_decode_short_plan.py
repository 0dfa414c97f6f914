"""Decode attention over heads on either side of the size up to which eight workgroups take one, and the final merge of more than eight
workgroups: by waves up to 64, through LDS beyond and for groups of 5 heads and more."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,G,rows", [(torch.bfloat16, 128, 1, 1536), (torch.bfloat16, 64, 4, 3072), (torch.bfloat16, 256, 2, 768),
                                            (torch.float32, 128, 4, 768), (torch.bfloat16, 128, 5, 2048), (torch.bfloat16, 64, 8, 3072), (torch.float32, 128, 6, 1024)])
def test_either_side_of_the_line(dtype, D, G, rows):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(rows + G)
    for n, eight in ((513, True), (rows - 1, True), (rows, True), (rows + 1, False)):
        Q = torch.randn((2, 2 * G, D), generator=g, device=dev).to(dtype)
        K, V = (torch.randn((2, 2, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
        ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(2, 2 * G, n, D), dtype=torch.uint8, device=dev)
        binding.l2kv_decode_workspace_init(ws)
        O, O8 = (torch.empty((2, 2 * G, D), device=dev) for _ in range(2))
        l2kv.l2kv_decode_attn(Q, K, V, O, ws)
        binding.l2kv_decode_attn_splits(Q, K, V, O8, ws, n_splits=8)
        if eight:
            assert torch.equal(O, O8)                       # the same plan: the same order of the sums
        q, k, v = Q.cpu().double(), K.cpu().double(), V.cpu().double()
        k, v = (x.repeat_interleave(G, dim=1) for x in (k, v))
        p = torch.softmax((k @ q[..., None])[..., 0] / math.sqrt(D), dim=-1)
        want = (p[..., None] * v).sum(dim=2)
        # fp32 sums of at most (n / 16 rows + the merges) terms of magnitude max |V| < 6 times weights that add up to 1
        assert (O.cpu().double() - want).abs().max() <= (n / 16 + 64) * 2.0 ** -24 * 6


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256), (torch.float32, 64), (torch.float32, 128)])
@pytest.mark.parametrize("G", [1, 3, 4, 5])
def test_merge_of_many_workgroups(dtype, D, G):
    if D == 256 and G > 4:
        pytest.skip("not a supported group")
    dev = torch.device("cuda:0")
    n = 4200
    g = torch.Generator(device=dev).manual_seed(D + G)
    Q = (2 * torch.randn((1, 3 * G, D), generator=g, device=dev)).to(dtype)
    K, V = (torch.randn((1, 3, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, 3 * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    q, k, v = Q.cpu().double(), K.cpu().double(), V.cpu().double()
    k, v = (x.repeat_interleave(G, dim=1) for x in (k, v))
    p = torch.softmax((k @ q[..., None])[..., 0] / math.sqrt(D), dim=-1)
    want = (p[..., None] * v).sum(dim=2)
    O = torch.empty((1, 3 * G, D), device=dev)
    for splits in (8, 9, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 66):
        for _ in range(2):                                  # the counters are left as they were found
            O.fill_(float("nan"))
            binding.l2kv_decode_attn_splits(Q, K, V, O, ws, n_splits=splits)
            assert (O.cpu().double() - want).abs().max() <= (n / 16 + 64) * 2.0 ** -24 * 6, splits


@pytest.mark.parametrize("dtype,D,G,heads,n,splits", [(torch.bfloat16, 128, 5, 3, 1615, 13), (torch.float32, 64, 8, 3, 1790, 14), (torch.bfloat16, 128, 5, 1, 1804, 14),
                                                      (torch.bfloat16, 128, 5, 3, 1804, 8), (torch.float32, 128, 6, 2, 929, 8), (torch.bfloat16, 128, 5, 12, 1615, 8),
                                                      (torch.bfloat16, 64, 5, 3, 2700, 8)])
def test_few_heads_of_large_groups(dtype, D, G, heads, n, splits):
    """Eight workgroups unless the longest of them reads much more than it would in more."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n)
    Q = torch.randn((1, heads * G, D), generator=g, device=dev).to(dtype)
    K, V = (torch.randn((1, heads, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    O, same, other = (torch.empty((1, heads * G, D), device=dev) for _ in range(3))
    l2kv.l2kv_decode_attn(Q, K, V, O, ws)
    binding.l2kv_decode_attn_splits(Q, K, V, same, ws, n_splits=splits)
    binding.l2kv_decode_attn_splits(Q, K, V, other, ws, n_splits=splits + 1)
    assert torch.equal(O, same) and not torch.equal(O, other)           # the same plan: the same order of the sums


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256), (torch.float32, 128)])
@pytest.mark.parametrize("G", [1, 4])
def test_merge_of_what_is_not_finite(dtype, D, G):
    """Values and scores that are not finite come out of the merge by waves as out of that of eight workgroups."""
    dev, n = torch.device("cuda:0"), 4200
    g = torch.Generator(device=dev).manual_seed(D + G)
    Q = (2 * torch.randn((1, 2 * G, D), generator=g, device=dev)).to(dtype)
    K, V = (torch.randn((1, 2, n, D), generator=g, device=dev).to(dtype) for _ in range(2))
    V[0, 0, 0, 3], V[0, 0, 2000, 5], V[0, 1, 10, 7] = -torch.inf, torch.nan, torch.inf
    K[0, 0, 2222] = torch.where(Q[0, 0] > 0, -torch.inf, torch.inf).to(dtype)          # -inf for the first query head, NaN for others
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, 2 * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    want, O = (torch.empty((1, 2 * G, D), device=dev) for _ in range(2))
    binding.l2kv_decode_attn_splits(Q, K, V, want, ws, n_splits=8)
    assert want[0, 0, 3] == -torch.inf and want[0, 0, 5].isnan() and (want[0, G:, 7] == torch.inf).all()
    for splits in (9, 16, 17, 24, 32, 47, 64):
        binding.l2kv_decode_attn_splits(Q, K, V, O, ws, n_splits=splits)
        finite = want.isfinite()
        assert torch.equal(O.isnan(), want.isnan()) and torch.equal(O[~finite & ~want.isnan()], want[~finite & ~want.isnan()])
        assert (O[finite] - want[finite]).abs().max() <= 2 * (n / 16 + 64) * 2.0 ** -24 * 6       # two orders of the sums
