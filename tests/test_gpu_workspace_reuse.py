"""One decode workspace, and the library's own scratch memory, under calls of different shapes one after the other: few heads in many
workgroups, whose partial results are the first behind the counters, then more heads, which need more counters."""
import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8, 8192), (70, 4, 900), (2, 1, 20000), (128, 1, 2048), (8, 4, 13108), (340, 4, 1536), (3, 2, 100), (200, 2, 2048)]     # heads, query heads each, rows


def operands(heads, G, n):
    g = torch.Generator(device="cuda:0").manual_seed(n + heads)
    Q = torch.randn((1, heads * G, 128), generator=g, device="cuda:0").to(torch.bfloat16)
    K, V = (torch.randn((1, heads, n, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    return Q, K, V


def workspace(nbytes):
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    binding.l2kv_decode_workspace_init(ws)
    return ws


def test_uniform():
    shared = workspace(max(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, 128) for heads, G, n in SHAPES))
    for heads, G, n in SHAPES * 2:
        Q, K, V = operands(heads, G, n)
        want, here, static = (torch.full((1, heads * G, 128), float("nan"), device="cuda:0") for _ in range(3))
        l2kv.l2kv_decode_attn(Q, K, V, want, workspace(l2kv.l2kv_decode_workspace_bytes(1, heads * G, n, 128)))
        l2kv.l2kv_decode_attn(Q, K, V, here, shared)
        binding.l2kv_decode_attn_static(Q, K, V, static)
        assert not want.isnan().any() and torch.equal(here, want) and torch.equal(static, want), (heads, G, n)


def test_ragged_between():
    """Sequences, with an order worked out inside the call, from the caller and in batch order, and a uniform call after each."""
    lens = [[9000, 30], [2500] * 40 + [300] * 30, [700] * 90, [40000], [2100, 5000, 2048] * 30]
    G, Hkv = 4, 2
    shared = workspace(max([l2kv.l2kv_decode_ragged_workspace_bytes(len(x), Hkv * G, max(x), 128) for x in lens] + [l2kv.l2kv_decode_workspace_bytes(1, 400, 2048, 128)]))
    for x in lens * 2:
        total = sum(x)
        g = torch.Generator(device="cuda:0").manual_seed(total)
        Q = torch.randn((len(x), Hkv * G, 128), generator=g, device="cuda:0").to(torch.bfloat16)
        K, V = (torch.randn((Hkv, total, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
        dev_lens = torch.tensor(x, dtype=torch.int32, device="cuda:0")
        slots = torch.cumsum(torch.tensor([0] + x), 0).cuda()
        order = torch.empty(len(x), dtype=torch.int32, device="cuda:0")
        l2kv.l2kv_length_order(dev_lens, order)
        for o in (None, order):
            want, here = (torch.full((len(x), Hkv * G, 128), float("nan"), device="cuda:0") for _ in range(2))
            for out, ws in ((want, workspace(l2kv.l2kv_decode_ragged_workspace_bytes(len(x), Hkv * G, max(x), 128))), (here, shared)):
                l2kv.l2kv_decode_attn_ragged(Q, K, V, dev_lens, slots, max(x), out, ws, seq_order=o)
            assert not want.isnan().any() and torch.equal(here, want), (x[:3], o is None)
        heads, n = 200, 2048
        Q, K, V = operands(heads, 2, n)
        want, here = (torch.full((1, heads * 2, 128), float("nan"), device="cuda:0") for _ in range(2))
        l2kv.l2kv_decode_attn(Q, K, V, want, workspace(l2kv.l2kv_decode_workspace_bytes(1, heads * 2, n, 128)))
        l2kv.l2kv_decode_attn(Q, K, V, here, shared)
        assert torch.equal(here, want)


def test_after_values_that_are_not_numbers():
    """Partial results that are NaN, with the sign set, where the next call has its counters."""
    g = torch.Generator(device="cuda:0").manual_seed(1)
    n, G = 9000, 4
    Q, K = (torch.randn(shape, generator=g, device="cuda:0") for shape in ((1, G, 128), (1, 1, n, 128)))
    V = torch.full((1, 1, n, 128), -1, dtype=torch.int32, device="cuda:0").view(torch.float32)
    shared = workspace(max(l2kv.l2kv_decode_workspace_bytes(*x, 128) for x in ((1, G, n), (1, 340 * 4, 1536))))
    O = torch.empty((1, G, 128), device="cuda:0")
    for heads, G2, rows in ((70, 4, 900), (128, 1, 2048), (340, 4, 1536)):
        l2kv.l2kv_decode_attn(Q, K, V, O, shared)
        binding.l2kv_decode_attn_static(Q, K, V, O)
        words = shared.view(torch.int32)[64:heads + 64]
        assert O.isnan().all() and ((words < 0) & (words >= -(1 << 22))).any()          # -1 .. 0xffc00000
        q, k, v = operands(heads, G2, rows)
        want, here, static = (torch.full((1, heads * G2, 128), float("nan"), device="cuda:0") for _ in range(3))
        l2kv.l2kv_decode_attn(q, k, v, want, workspace(l2kv.l2kv_decode_workspace_bytes(1, heads * G2, rows, 128)))
        l2kv.l2kv_decode_attn(q, k, v, here, shared)
        binding.l2kv_decode_attn_static(q, k, v, static)
        assert not want.isnan().any() and torch.equal(here, want) and torch.equal(static, want)
        assert not shared.view(torch.int32)[:heads].any()


def test_after_values_whose_bits_are_small_numbers():
    """Values of a few 2^-149, whose partial sums have the bits of a count of workgroups: those are not left in the workspace, and larger
    ones are what they were."""
    g = torch.Generator(device="cuda:0").manual_seed(2)
    n, G = 9000, 4
    Q, K = (torch.randn(shape, generator=g, device="cuda:0") for shape in ((1, G, 128), (1, 1, n, 128)))
    V = (torch.randint(0, 3, (1, 1, n, 128), generator=g, device="cuda:0", dtype=torch.int32) * (torch.rand((1, 1, n, 1), generator=g, device="cuda:0") < 0.02)).to(torch.int32)
    V[..., 64:] += 1 << 23                                               # normal numbers
    V = V.view(torch.float32)
    shared = workspace(max(l2kv.l2kv_decode_workspace_bytes(*x, 128) for x in ((1, G, n), (1, 340 * 4, 1536))))
    O = torch.empty((1, G, 128), device="cuda:0")
    l2kv.l2kv_decode_attn(Q, K, V, O, shared)
    binding.l2kv_decode_attn_static(Q, K, V, O)
    assert torch.all((O[..., 64:].double() / 2.0 ** -126 - 1).abs() < 1e-3) and torch.all(O[..., :64].abs() <= 2.0 ** -141)
    for heads, G2, rows in ((70, 4, 900), (128, 1, 2048), (340, 4, 1536)):
        l2kv.l2kv_decode_attn(Q, K, V, O, shared)
        binding.l2kv_decode_attn_static(Q, K, V, O)
        words = shared.view(torch.int32)
        assert (words[64:heads + 64] >= 1 << 22).any() and not ((words > 0) & (words < 256)).any()
        q, k, v = operands(heads, G2, rows)
        want, here, static = (torch.full((1, heads * G2, 128), float("nan"), device="cuda:0") for _ in range(3))
        l2kv.l2kv_decode_attn(q, k, v, want, workspace(l2kv.l2kv_decode_workspace_bytes(1, heads * G2, rows, 128)))
        l2kv.l2kv_decode_attn(q, k, v, here, shared)
        binding.l2kv_decode_attn_static(q, k, v, static)
        assert not want.isnan().any() and torch.equal(here, want) and torch.equal(static, want)


def test_after_an_order_of_its_own():
    """The order that a ragged call works out for itself stays in the workspace: its numbers are no counts."""
    n_seq, Hkv, G, rows = 300, 1, 1, 2048
    ws = workspace(l2kv.l2kv_decode_ragged_workspace_bytes(n_seq, Hkv * G, rows, 128))
    g = torch.Generator(device="cuda:0").manual_seed(3)
    lens = torch.randint(1, 40, (n_seq,), generator=g, device="cuda:0", dtype=torch.int32)
    slots = torch.zeros(n_seq + 1, dtype=torch.int64, device="cuda:0")
    slots[1:] = torch.cumsum(lens, 0)
    total = max(rows, int(slots[-1]))
    Q = torch.randn((n_seq, 1, 128), generator=g, device="cuda:0").to(torch.bfloat16)
    K, V = (torch.randn((Hkv, total, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    order = torch.empty(n_seq, dtype=torch.int32, device="cuda:0")
    l2kv.l2kv_length_order(lens, order)
    want, here = (torch.full((n_seq, 1, 128), float("nan"), device="cuda:0") for _ in range(2))
    l2kv.l2kv_decode_attn_ragged(Q, K, V, lens, slots, rows, want, ws, seq_order=order)
    l2kv.l2kv_decode_attn_ragged(Q, K, V, lens, slots, rows, here, ws)
    assert not want.isnan().any() and torch.equal(here, want) and torch.equal(torch.sort(order).values, torch.arange(n_seq, dtype=torch.int32, device="cuda:0"))
    words = ws.view(torch.int32)
    assert not ((words > 0) & (words < 256)).any()
