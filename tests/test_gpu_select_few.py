"""The search of heads of at most 2048 tokens, in 2048 bins: few keys of a bin compared by every wave (up to 8), more through LDS (up to 256), and
bins that are divided again; against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_11430_amd as l2kv

pytestmark = pytest.mark.gpu


def keys(kind, T, rng):
    if kind == "norms":
        return (128 * np.exp(rng.standard_normal((4, T)))).astype(np.float32)
    if kind == "zero row":
        x = (128 + rng.standard_normal((4, T))).astype(np.float32)
        x[:, T // 2] = 0.0
        return x
    if kind == "bits":
        return rng.integers(0, 2 ** 32, (4, T), dtype=np.uint64).astype(np.uint32).view(np.float32)
    each = int(kind)                                                   # so many neighbouring bit patterns, and far from them the others
    near = np.uint32(0x43000000) + rng.permutation(each).astype(np.uint32)
    x = np.concatenate([near[:T], (np.uint32(0x10000000) + rng.integers(0, 1 << 30, max(0, T - each)).astype(np.uint32))])
    return np.stack([rng.permutation(x) for _ in range(4)]).view(np.float32)


@pytest.mark.parametrize("kind", ["norms", "zero row", "bits", "7", "8", "9", "64", "65", "255", "256", "257", "900"])
@pytest.mark.parametrize("T", [1, 2, 9, 63, 1000, 1024, 1025, 2047, 2048, 2049])
def test_matches_the_oracle(T, kind):
    x = keys(kind, T, np.random.default_rng(T))
    nd = torch.from_numpy(x).cuda()
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    inside = int((np.sort(x.view(np.uint32)[0]) < 0x43000000).sum())    # the first of the neighbours and those around it
    for k in sorted({max(1, min(T, v)) for v in (1, T // 10, T // 2, T, inside, inside + 1, inside + 5, inside + 200)}):
        for mode in (l2kv.L2KV_KEEP_LOWEST, l2kv.L2KV_KEEP_HIGHEST):
            idx = torch.full((4, k), -7, dtype=torch.int32, device="cuda")
            l2kv.l2kv_select_k(nd, k, mode, idx, None, ws)
            np.testing.assert_array_equal(idx.cpu().numpy(), oracle.select(x, k, mode), err_msg="k=%d mode=%d" % (k, mode))
