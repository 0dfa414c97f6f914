"""Blocks of positions of a share of the losses and the registers that hold them (csrc/position_blocks.hpp), on the host."""
import ctypes as C
import shutil
import subprocess

import pytest

from paper_2406_11430_amd import build

SOURCE = """
#include <hip/hip_runtime.h>
#include "position_blocks.hpp"
#define SLOTS(n) extern "C" void slots_##n(unsigned blocks, unsigned share, unsigned shares, unsigned* out) { \\
    const l2kv::PositionBlocks<n> b(blocks, share, shares); \\
    for (unsigned j = 0; j < n; ++j) out[j] = b.in_slot(j); \\
    for (unsigned e = 0; e < 32; ++e) out[n + e] = b.has(e); \\
}
SLOTS(8) SLOTS(12) SLOTS(16) SLOTS(20)
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which(build.hipcc()) is None:
        pytest.skip("no hipcc")
    where = tmp_path_factory.mktemp("blocks")
    (where / "blocks.hip").write_text(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + build.CSRC, str(where / "blocks.hip"),
                    "-o", str(where / "blocks.so")], check=True, capture_output=True)
    return C.CDLL(str(where / "blocks.so"))


@pytest.mark.parametrize("slots", [8, 12, 16, 20])
def test_every_block_once_and_none_past_the_head(lib, slots):
    out = (C.c_uint * (slots + 32))()
    for blocks in range(2, 33):
        for shares in range((blocks + slots - 1) // slots, blocks + 1):
            taken = []
            for share in range(shares):
                getattr(lib, "slots_%d" % slots)(blocks, share, shares, out)
                mine = [e for e in range(32) if out[slots + e]]
                assert mine and all(out[e % slots] == e for e in mine)
                assert all(out[j] in mine for j in range(slots)), (blocks, share, shares)     # what is fetched for nothing, too
                taken += mine
            assert taken == list(range(blocks))
