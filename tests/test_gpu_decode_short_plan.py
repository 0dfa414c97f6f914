"""Decode attention over heads on either side of the size up to which eight workgroups take one."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,G,rows", [(torch.bfloat16, 128, 1, 2048), (torch.bfloat16, 64, 4, 4096), (torch.bfloat16, 256, 2, 1024),
                                            (torch.float32, 128, 4, 1024), (torch.bfloat16, 128, 5, 2048), (torch.bfloat16, 64, 8, 3072), (torch.float32, 128, 6, 1024)])
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
