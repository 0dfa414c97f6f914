"""The launch shapes of the selection at the lengths where they change: one workgroup per head with
its keys in registers, re-read from memory, and several workgroups per head through the workspace
(chosen by the workspace size: 256 bytes always mean one workgroup per head)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_11430_amd as l2kv

pytestmark = pytest.mark.gpu


def keys(kind, n, T, rng):
    if kind == "norms":
        x = (rng.standard_normal((n, T)) ** 2 * np.exp(rng.standard_normal((n, T)))).astype(np.float32)
    elif kind == "equal":
        x = np.full((n, T), 3.25, np.float32)
    elif kind == "padded":                    # most rows zero: the k-th key is among the ties or just past them
        x = np.where(rng.random((n, T)) < 0.6, 0.0, rng.random((n, T))).astype(np.float32)
    else:                                     # any bit pattern, the largest one (the padding's) among them
        x = rng.integers(0, 2 ** 32, (n, T), dtype=np.uint64).astype(np.uint32)
        x[:, rng.integers(0, T, T // 3)] = 0xffffffff
        x = x.view(np.float32)
    return np.ascontiguousarray(x)


@pytest.mark.parametrize("kind", ["norms", "equal", "padded", "bits"])
@pytest.mark.parametrize("n,T", [(3, 1), (2, 1024), (2, 1025), (3, 8193), (2, 32768), (1, 32769), (5, 40001),
                                 (1, 65537), (32, 65536), (2, 131072), (33, 70001)])
def test_every_launch_shape_matches_the_oracle(n, T, kind):
    x = keys(kind, n, T, np.random.default_rng(n * 100003 + T))
    nd = torch.from_numpy(x).cuda()
    full = l2kv.l2kv_select_workspace_bytes(n, T)
    assert (full > 256) == (T > 32768 and n <= min(64, T // 2048))
    for k in sorted({1, (T + 1) // 2, max(1, T // 10), T}):
        for mode in (l2kv.L2KV_KEEP_LOWEST, l2kv.L2KV_KEEP_HIGHEST):
            want = oracle.select(x, k, mode)
            for size in sorted({256, full - 16 if full > 256 else 256, full}):
                ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
                idx = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
                cnt = torch.zeros(n, dtype=torch.int32, device="cuda")
                l2kv.l2kv_select_k(nd, k, mode, idx, cnt, ws)
                np.testing.assert_array_equal(idx.cpu().numpy(), want, err_msg="%s k=%d mode=%d ws=%d" % (kind, k, mode, size))
                assert (cnt == k).all()


def test_split_heads_under_graph_capture():
    """Three kernels and a workspace instead of one kernel: replays on new keys match eager calls."""
    n, T, k = 4, 50000, 20000
    rng = np.random.default_rng(5)
    nd = torch.empty((n, T), dtype=torch.float32, device="cuda")
    idx = torch.empty((n, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(l2kv.l2kv_select_workspace_bytes(n, T), dtype=torch.uint8, device="cuda")
    nd.copy_(torch.from_numpy(keys("norms", n, T, rng)))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        l2kv.l2kv_select_k(nd, k, l2kv.L2KV_KEEP_LOWEST, idx, None, ws)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        l2kv.l2kv_select_k(nd, k, l2kv.L2KV_KEEP_LOWEST, idx, None, ws)
    for kind in ("norms", "padded", "norms"):
        x = keys(kind, n, T, rng)
        nd.copy_(torch.from_numpy(x))
        torch.cuda.synchronize()
        idx.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx.cpu().numpy(), oracle.select(x, k, l2kv.L2KV_KEEP_LOWEST))


def expected(x, k):
    """By a stable sort of the bit patterns on the device, for heads too long for the oracle."""
    by_key = torch.sort(x.view(torch.int32).to(torch.int64) & 0xFFFFFFFF, dim=-1, stable=True).indices[:, :k]
    return torch.sort(by_key, dim=-1).values.to(torch.int32)


# chunks of 32768 keys, the longest with 16-bit counts; of 36864 and 524288 with 32-bit ones; 512 chunks of one head
@pytest.mark.parametrize("kind", ["norms", "equal", "padded", "bits"])
@pytest.mark.parametrize("n,T", [(64, 262144), (64, 262145), (64, 280001), (8, 4194304), (1, 4194303)])
def test_long_chunks(n, T, kind):
    g = torch.Generator(device="cuda").manual_seed(T)
    u = torch.rand((n, T), generator=g, device="cuda")
    if kind == "norms":
        x = torch.exp(torch.randn((n, T), generator=g, device="cuda"))
    elif kind == "equal":
        x = torch.full((n, T), 3.25, device="cuda")
    elif kind == "padded":
        x = torch.where(u < 0.6, torch.zeros_like(u), u)
    else:
        x = torch.randint(-2 ** 31, 2 ** 31, (n, T), generator=g, device="cuda").to(torch.int32)
        x[u < 0.3] = -1
        x = x.view(torch.float32)
    full = l2kv.l2kv_select_workspace_bytes(n, T)
    assert full > 4 * n * T
    for k in (1, T // 10, T // 2, T):
        ws = torch.full((full,), 0xA5, dtype=torch.uint8, device="cuda")
        idx = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
        l2kv.l2kv_select_k(x, k, l2kv.L2KV_KEEP_LOWEST, idx, None, ws)
        assert torch.equal(idx, expected(x, k)), k


def test_equal_keys_do_not_grow_with_the_square_of_the_length():
    """Every workgroup of a head goes over all of its candidates, which are all keys where all are equal: 64 heads of
    1M took 14 times as long as distinct ones while the number of workgroups grew with the length."""
    n, T, k = 64, 1 << 20, 1 << 18
    ws = torch.empty(l2kv.l2kv_select_workspace_bytes(n, T), dtype=torch.uint8, device="cuda")
    idx = torch.empty((n, k), dtype=torch.int32, device="cuda")
    took = []
    for x in (torch.exp(torch.randn((n, T), device="cuda")), torch.full((n, T), 3.25, device="cuda")):
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                l2kv.l2kv_select_k(x, k, l2kv.L2KV_KEEP_LOWEST, idx, None, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
    assert took[1] <= 9 * took[0], took
