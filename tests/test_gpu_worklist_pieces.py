"""Ragged decode attention over work lists whose sequences are cut into pieces because some are much longer than a workgroup's
share of the whole: against the same launch with one workgroup per sequence."""
import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


# pairs: pieces of their own for all; just not; three; two; whole
@pytest.mark.parametrize("n_seq,Hkv,G", [(1, 1, 4), (8, 4, 1), (8, 8, 4), (12, 8, 4), (16, 8, 2), (20, 8, 4), (24, 8, 6), (30, 8, 4), (31, 8, 1),
                                         (40, 8, 4), (64, 8, 4)])
def test_pieces(n_seq, Hkv, G):
    dev, D = torch.device("cuda:0"), 128
    g = torch.Generator(device="cpu").manual_seed(n_seq)
    lens = torch.randint(0, 2600, (n_seq,), generator=g)
    lens[0] = 2599
    off = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lens + 1, 0)])
    slots = int(off[-1])
    gd = torch.Generator(device=dev).manual_seed(n_seq)
    K, V = (torch.randn((Hkv, slots, D), generator=gd, device=dev).bfloat16() for _ in range(2))
    Q = torch.randn((n_seq, Hkv * G, D), generator=gd, device=dev).bfloat16()
    lens_d, off_d = lens.to(torch.int32).to(dev), off.to(dev)
    order = torch.empty((n_seq,), dtype=torch.int32, device=dev)
    l2kv.l2kv_length_order(lens_d, order)
    ws = torch.empty(l2kv.l2kv_decode_ragged_workspace_bytes(n_seq, Hkv * G, 2600, D), dtype=torch.uint8, device=dev)
    binding.l2kv_decode_workspace_init(ws)
    O, one = (torch.full((n_seq, Hkv * G, D), float("nan"), device=dev) for _ in range(2))
    l2kv.l2kv_decode_attn_ragged(Q, K, V, lens_d, off_d, 2600, one, ws, n_splits=1)           # a grid, in batch order
    for _ in range(3):                                                                      # the list is left as it was found
        O.fill_(float("nan"))
        l2kv.l2kv_decode_attn_ragged(Q, K, V, lens_d, off_d, 2600, O, ws, seq_order=order)
        # two orders of fp32 sums of up to 2600 / 16 terms, weights that add up to 1, values below 6
        assert (O - one).abs().max() <= 2 * (2600 / 16 + 64) * 2.0 ** -24 * 6
