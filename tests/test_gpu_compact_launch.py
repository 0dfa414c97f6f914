"""Compaction launches: row sizes and counts around a wave's share of rows, more heads than one
launch takes in its second dimension, and ragged batches whose sequences begin and end inside a wave."""
import numpy as np
import pytest
import torch

import paper_2406_11430_amd as l2kv

pytestmark = pytest.mark.gpu

ROWS = [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 128)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


def bits(shape, dtype, g, dev):
    """Random bit patterns: the calls copy bytes."""
    words = torch.randint(-2**31, 2**31 - 1, (*shape[:-1], shape[-1] * dtype.itemsize // 4), generator=g, dtype=torch.int64)
    return words.to(torch.int32).to(dev).view(dtype)


def same(a, b):
    return torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32))


@pytest.mark.parametrize("dtype,D", ROWS)
# 64 (short rows 128) rows of K and V to a workgroup from that many rows on, up to 16 MB (1024 workgroups of 256-byte rows);
# else 16 (32) of either
@pytest.mark.parametrize("heads,T,k", [(1, 1, 1), (3, 40, 15), (3, 40, 16), (2, 70, 33), (70001, 2, 1), (3, 70, 64), (2, 140, 65),
                                       (1, 200, 127), (5, 200, 129), (1024, 130, 64), (1025, 130, 64), (512, 130, 128), (513, 260, 129)])
@pytest.mark.parametrize("with_v", [True, False])
def test_compact(dev, dtype, D, heads, T, k, with_v):
    g = torch.Generator().manual_seed(heads + T + k)
    K = bits((heads, T, D), dtype, g, dev)
    V = bits((heads, T, D), dtype, g, dev) if with_v else None
    idx = torch.argsort(torch.rand((heads, T), generator=g), dim=-1)[:, :k].sort(-1).values.to(torch.int32).to(dev)
    Kc = torch.empty((heads, k, D), dtype=dtype, device=dev)
    Vc = torch.empty_like(Kc) if with_v else None
    l2kv.l2kv_compact(K, V, idx, Kc, Vc)
    at = idx.long()[..., None].expand(heads, k, D)
    assert same(Kc, torch.gather(K, 1, at))
    assert not with_v or same(Vc, torch.gather(V, 1, at))


# 1, 2, 64, 65 and 4097 sequences: one, two and three steps of the owner search; runs of empty sequences around
# the 64 that a row looks through at once
@pytest.mark.parametrize("dtype,D", ROWS)
@pytest.mark.parametrize("n_seq,longest,planes,empty", [(1, 200, 2, 0), (2, 9, 1, 0), (64, 6, 3, 0), (65, 40, 2, 0), (4097, 5, 2, 0),
                                                        (3, 4, 65539, 0), (600, 5, 2, 62), (600, 5, 2, 64), (600, 9, 1, 131),
                                                        (300, 3, 1, 290)])
def test_compact_ragged(dev, dtype, D, n_seq, longest, planes, empty):
    rng = np.random.default_rng(n_seq)
    kept = rng.integers(0, longest + 1, n_seq)                       # empty sequences too
    if empty:
        for first in range(3, n_seq, empty + 5):
            kept[first:first + empty] = 0
    kept[0] = longest
    length = kept + rng.integers(0, 4, n_seq)
    room = kept + rng.integers(0, 3, n_seq)
    offs = [np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (length, kept, room)]
    in_off, out_off, slot_off = (torch.from_numpy(o).to(dev) for o in offs)
    total, total_kept, slots = (int(o[-1]) for o in offs)
    local = np.concatenate([np.sort(rng.permutation(l)[:c]) for l, c in zip(length, kept)]).astype(np.int64)
    seq = np.repeat(np.arange(n_seq), kept)
    src = torch.from_numpy(offs[0][seq] + local).to(dev)
    dst = torch.from_numpy(offs[2][seq] + np.arange(total_kept) - offs[1][seq]).to(dev)
    g = torch.Generator().manual_seed(n_seq)
    K, V = bits((planes, total, D), dtype, g, dev), bits((planes, total, D), dtype, g, dev)
    norms = torch.rand((planes, total), generator=g).to(dev)
    idx = torch.from_numpy(local.astype(np.int32)).to(dev).expand(planes, total_kept).contiguous()
    Kc = torch.zeros((planes, slots, D), dtype=dtype, device=dev)
    Vc = torch.zeros_like(Kc)
    norms_c = torch.zeros((planes, slots), device=dev)
    pos_c = torch.full((planes, slots), -1, dtype=torch.int32, device=dev)
    l2kv.l2kv_compact_ragged(K, V, norms, idx, in_off, out_off, int(kept.max()), slot_off, Kc, Vc, norms_c, pos_c)
    for got, x in ((Kc, K), (Vc, V)):
        want = torch.zeros_like(got)
        want[:, dst] = x[:, src]
        assert same(got, want)
    want = torch.zeros_like(norms_c)
    want[:, dst] = norms[:, src]
    assert torch.equal(norms_c, want)
    want = torch.full_like(pos_c, -1)
    want[:, dst] = idx
    assert torch.equal(pos_c, want)
