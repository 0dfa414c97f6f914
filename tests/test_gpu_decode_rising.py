"""Scores that rise from row to row, so that every tile moves the running maximum, far from zero: the weights of the rows before and after
each move belong together."""
import math

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


# one head on the vector unit and several, q.k and p.V on the matrix unit; one workgroup and a few; rows of pairs
@pytest.mark.parametrize("dtype,D,G", [(torch.float32, 64, 1), (torch.float32, 128, 8), (torch.bfloat16, 64, 4), (torch.bfloat16, 128, 1), (torch.bfloat16, 128, 6), (torch.bfloat16, 128, 8),
                                       (torch.bfloat16, 256, 4)])
@pytest.mark.parametrize("n_splits", [1, 2, 12])
def test_rising_scores(dtype, D, G, n_splits):
    dev, heads, n = torch.device("cuda:0"), 16, 1024
    g = torch.Generator(device=dev).manual_seed(D + G)
    V = torch.randn((1, heads, n, D), generator=g, device=dev).to(dtype)
    K = torch.zeros((1, heads, n, D), device=dev)
    K[..., 5] = 200.0
    K[..., 6] = torch.arange(n, device=dev) // 4 / 64.0                # up to 4 more; 256 values, exact in 8 bits, as are all products and sums
    Q = torch.zeros((1, heads * G, D), device=dev)
    Q[..., 5] = Q[..., 6] = 8.0
    Q, K = Q.to(dtype), K.to(dtype)
    ws = torch.empty(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    O = torch.empty((1, heads * G, D), device=dev)
    binding.l2kv_decode_attn_splits(Q, K, V, O, ws, n_splits=n_splits)
    p = torch.softmax(8.0 * (K[..., 5].double() + K[..., 6].double()) / math.sqrt(D), dim=-1)
    want = (p[..., None] * V.double()).sum(dim=2).repeat_interleave(G, dim=1)
    # Sums of 64 terms a lane, 16 to 32 lanes and 12 workgroups, each rounded by 2^-25 of itself in the mean square or less, and weights
    # 2^x with |x| < 47 off by 2^-24 |x| ln 2, the lowest of which count for nothing: e^-x |x| < 0.4.  Together below 2^-21 of the result's size.
    # (A factor off by the rounding of 288 alone, 2^-16, shows 30 times as much.)
    assert (O.double() - want).norm() <= 2.0 ** -21 * want.norm()
