"""Ordered ragged batches are cut by the lengths the kernel finds, not by the caller's bound of them."""
import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu

BATCHES = {"alike": ([4000] * 24, 1), "alike, few": ([4000] * 12, 2), "one long": ([8000] + [500] * 23, 7), "some long": ([500] * 10 + [8000] * 4 + [500] * 17, 4),
           "mixed": ([500 + 170 * i for i in range(24)], 3), "compute units": ([3000, 2100, 2500], 8)}


@pytest.mark.parametrize("name", BATCHES)
@pytest.mark.parametrize("G", [1, 4, 6])
def test_bound(name, G):
    lens, pieces = BATCHES[name]
    dev, D, Hkv, n, longest = torch.device("cuda:0"), 128, 8, len(lens), max(lens)
    off = torch.cumsum(torch.tensor([0] + lens), 0)
    g = torch.Generator(device=dev).manual_seed(n)
    K, V = (torch.randn((Hkv, int(off[-1]), D), generator=g, device=dev).bfloat16() for _ in range(2))
    Q = torch.randn((n, Hkv * G, D), generator=g, device=dev).bfloat16()
    lens_d, off_d = torch.tensor(lens, dtype=torch.int32, device=dev), off.to(dev)
    order = torch.empty((n,), dtype=torch.int32, device=dev)
    l2kv.l2kv_length_order(lens_d, order)

    def run(bound, order, n_splits=0):
        ws = torch.empty(l2kv.l2kv_decode_ragged_workspace_bytes(n, Hkv * G, bound, D), dtype=torch.uint8, device=dev)
        binding.l2kv_decode_workspace_init(ws)
        O = torch.full((n, Hkv * G, D), float("nan"), device=dev)
        for _ in range(2):
            l2kv.l2kv_decode_attn_ragged(Q, K, V, lens_d, off_d, bound, O, ws, n_splits=n_splits, seq_order=order)
        assert not ws[:4 * (n * Hkv + 2)].any()
        return O

    want = run(longest, order, pieces)                                # cut into as many by the caller: the same order of the sums
    assert (want - run(longest, order, 1)).abs().max() <= 2 * (longest / 16 + 64) * 2.0 ** -24 * 6
    for bound in ({longest, int(1.3 * longest), 2 * longest} if name != "compute units" else {longest}):
        bound = min(bound, int(off[-1]))
        assert torch.equal(run(bound, order), want)
        assert torch.equal(run(bound, None), want)                    # an order of the library's own
    # an order that no longer has the longest in front steers only the cut
    for stale in (order.flip(0).contiguous(), order.roll(1)):
        assert (run(longest, stale) - want).abs().max() <= 2 * (longest / 16 + 64) * 2.0 ** -24 * 6


def test_first_in_the_order_is_empty():
    dev, D, Hkv = torch.device("cuda:0"), 128, 8
    lens, off = torch.tensor([0, 2500, 2200], dtype=torch.int32, device=dev), torch.tensor([0, 8, 2508, 4708], device=dev)
    g = torch.Generator(device=dev).manual_seed(3)
    K, V = (torch.randn((Hkv, 4708, D), generator=g, device=dev).bfloat16() for _ in range(2))
    Q = torch.randn((3, Hkv, D), generator=g, device=dev).bfloat16()
    for Hk in (Hkv, 1):                                               # more and fewer pairs than the load matters for
        ws = torch.empty(l2kv.l2kv_decode_ragged_workspace_bytes(3, Hk, 2500, D), dtype=torch.uint8, device=dev)
        binding.l2kv_decode_workspace_init(ws)
        out = []
        for order in ([0, 1, 2], [1, 2, 0]):
            O = torch.full((3, Hk, D), float("nan"), device=dev)
            l2kv.l2kv_decode_attn_ragged(Q[:, :Hk].contiguous(), K[:Hk].contiguous(), V[:Hk].contiguous(), lens, off, 2500, O, ws,
                                         seq_order=torch.tensor(order, dtype=torch.int32, device=dev))
            out.append(O)
        assert (out[0][0] == 0).all() and (out[0] - out[1]).abs().max() <= 2 * (2500 / 16 + 64) * 2.0 ** -24 * 6
