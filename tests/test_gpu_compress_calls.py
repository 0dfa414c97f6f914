"""l2kv_compress through the C entry point, with what the Python function does not pass: heads further apart than
their rows, slabs over every kind of launch (one for the shortest heads, two, three, and the selection that shares
long heads among workgroups), and a workspace that must not be touched."""
import numpy as np
import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible: the gpu tests need a real MI355X")
    l2kv.lib()
    return torch.device("cuda:0")


def rows(shape, dtype, g, dev):
    x = torch.randn(shape, generator=g, device=dev) * torch.exp(0.5 * torch.randn(shape[:-1] + (1,), generator=g, device=dev))
    x[:, ::7] = x[:, :1].clone()                                               # ties
    return x.to(dtype)


def expected(K, V, k):
    n, T, D = K.shape
    norms = torch.empty((n, T), device=K.device)
    l2kv.l2kv_norms(K, norms)
    idx = torch.sort(torch.sort(norms.view(torch.int32), dim=-1, stable=True).indices[:, :k], dim=-1).values
    take = idx[..., None].expand(n, k, D)
    return norms, idx.to(torch.int32), torch.gather(K, 1, take), torch.gather(V, 1, take)


def compress(K, V, gap, ratio, slab, ws):
    """K, V [n][T][D] laid out with `gap` more rows behind every head."""
    n, T, D = K.shape
    k = l2kv.l2kv_keep_count(T, ratio)
    wide = [torch.full((n, T + gap, D), 7.0, dtype=K.dtype, device=K.device) for _ in range(2)]
    for w, x in zip(wide, (K, V)):
        w[:, :T] = x
    out = [torch.full((n, T), -1.0, device=K.device), torch.full((n, k), -1, dtype=torch.int32, device=K.device),
           torch.zeros((n, k, D), dtype=K.dtype, device=K.device), torch.zeros((n, k, D), dtype=K.dtype, device=K.device)]
    dt = binding.L2KV_F32 if K.dtype == torch.float32 else binding.L2KV_BF16
    status = binding.lib().l2kv_compress(wide[0].data_ptr(), wide[1].data_ptr(), dt, n, T, D, (T + gap) * D, ratio, slab,
                                         *[o.data_ptr() for o in out], ws.data_ptr(), ws.numel(),
                                         torch.cuda.current_stream().cuda_stream)
    assert status == 0
    return out


# T: one launch up to 1024, two up to 4096, three, selection shared among workgroups beyond 32768
@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256), (torch.float32, 128)])
@pytest.mark.parametrize("heads,T,ratio", [(5, 1, 1.0), (5, 700, 0.5), (3, 1024, 0.9), (5, 3000, 0.3), (3, 8193, 0.5), (5, 33000, 0.5)])
@pytest.mark.parametrize("gap,slab", [(0, 0), (3, 0), (0, 1), (1, 2), (5, 4), (2, 5)])
def test_strides_and_slabs(dev, dtype, D, heads, T, ratio, gap, slab):
    g = torch.Generator(device=dev).manual_seed(T + heads)
    K, V = rows((heads, T, D), dtype, g, dev), torch.randn((heads, T, D), generator=g, device=dev).to(dtype)
    ws = torch.empty(256, dtype=torch.uint8, device=dev)
    for got, want in zip(compress(K, V, gap, ratio, slab, ws), expected(K, V, l2kv.l2kv_keep_count(T, ratio))):
        assert torch.equal(got, want)


# 1/32: the kept rows of 128 bytes are as large as the list of the selection; below, one workgroup per head selects
@pytest.mark.parametrize("D,ratio", [(64, 0.001), (64, 0.031), (64, 1 / 32), (64, 0.0313), (64, 0.05), (128, 0.015), (128, 0.016),
                                     (256, 0.0078), (256, 0.0079), (128, 1.0)])
@pytest.mark.parametrize("heads,T", [(2, 32769), (8, 60000), (1, 131072)])
def test_workspace_is_not_touched(dev, D, ratio, heads, T):
    """Calls may share it, also on streams that run at the same time: a selection that shares long heads among
    workgroups passes its counts and lists through the outputs."""
    g = torch.Generator(device=dev).manual_seed(T + D)
    K = rows((heads, T, D), torch.bfloat16, g, dev)
    V = torch.randn((heads, T, D), generator=g, device=dev).to(torch.bfloat16)
    ws = torch.randint(0, 256, (l2kv.l2kv_select_workspace_bytes(heads, T),), dtype=torch.uint8, device=dev, generator=g)
    before = ws.clone()
    for got, want in zip(compress(K, V, 0, ratio, 0, ws), expected(K, V, l2kv.l2kv_keep_count(T, ratio))):
        assert torch.equal(got, want)
    assert torch.equal(ws, before)


def test_two_streams_share_a_workspace(dev):
    heads, T, D, ratio = 4, 100000, 128, 0.3
    g = torch.Generator(device=dev).manual_seed(1)
    ws = torch.empty(l2kv.l2kv_select_workspace_bytes(heads, T), dtype=torch.uint8, device=dev)
    k = l2kv.l2kv_keep_count(T, ratio)
    streams = [torch.cuda.Stream() for _ in range(2)]
    calls = []
    for _ in streams:
        K = rows((heads, T, D), torch.bfloat16, g, dev)
        V = torch.randn((heads, T, D), generator=g, device=dev).to(torch.bfloat16)
        out = [torch.empty((heads, T), device=dev), torch.empty((heads, k), dtype=torch.int32, device=dev),
               torch.empty((heads, k, D), dtype=torch.bfloat16, device=dev), torch.empty((heads, k, D), dtype=torch.bfloat16, device=dev)]
        calls.append((K, V, out, expected(K, V, k)))
    torch.cuda.synchronize()
    for _ in range(20):
        for s, (K, V, out, _) in zip(streams, calls):
            l2kv.l2kv_compress(K, V, ratio, *out, ws, stream=s)
    torch.cuda.synchronize()
    for _, _, out, want in calls:
        for got, w in zip(out, want):
            assert torch.equal(got, w)
