"""Selection whose threshold lies in a bin of a given number of keys: those that every wave compares by itself, whole and broken groups of
sixteen, a full list; distinct and tied."""
import numpy as np
import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [512, 2048, 4000, 9000])
@pytest.mark.parametrize("listed", [1, 8, 9, 15, 16, 17, 31, 32, 33, 47, 240, 255, 256, 257])
def test_listed(T, listed):
    rng = np.random.default_rng(T + listed)
    low = np.float32(1.0).view(np.uint32)
    # the range of the keys makes bins of 2^17 or 2^16 bit patterns, of which one holds the keys that are listed
    span, base = 167 << 20, 100 << 17
    heads = []
    for kind in range(4):
        within = [np.arange(listed), rng.integers(0, 1 << 15, listed), rng.integers(0, 5, listed), np.zeros(listed)][kind].astype(np.uint32)
        bits = np.concatenate([[low, low + np.uint32(span)], low + np.uint32(base) + within, low + np.uint32(base - (1 << 20)) + rng.integers(0, 1 << 18, 100).astype(np.uint32),
                               low + np.uint32(base + (1 << 20)) + rng.integers(0, 1 << 26, T - listed - 102).astype(np.uint32)]).astype(np.uint32)
        heads.append(rng.permutation(bits))
    bits = np.stack(heads)
    norms = torch.from_numpy(bits.view(np.float32).copy()).cuda()
    ws = torch.empty(max(16, l2kv.l2kv_select_workspace_bytes(4, T)), dtype=torch.uint8, device="cuda:0")
    order = np.argsort(bits, axis=1, kind="stable")
    for wanted in sorted({1, (listed + 1) // 2, listed}):
        k = 101 + wanted                                              # the lowest and the hundred before the bin
        kept = torch.empty((4, k), dtype=torch.int32, device="cuda:0")
        binding.l2kv_select_k(norms, k, binding.L2KV_KEEP_LOWEST, kept, None, ws)
        assert np.array_equal(kept.cpu().numpy(), np.sort(order[:, :k], axis=1)), (T, listed, wanted)
