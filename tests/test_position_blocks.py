"""Shares of a head whose scores are ranked (csrc/rank_shares.hpp), the blocks of positions each adds up and the registers that hold them
(csrc/position_blocks.hpp), on the host."""
import ctypes as C
import shutil
import subprocess

import pytest

from paper_2406_11430_amd import build

SOURCE = """
#include <hip/hip_runtime.h>
#include "position_blocks.hpp"
#include "rank_shares.hpp"
#define SLOTS(n) extern "C" void slots_##n(unsigned blocks, unsigned share, unsigned shares, unsigned* out) { \\
    const l2kv::PositionBlocks<n> b(blocks, share, shares); \\
    for (unsigned j = 0; j < n; ++j) out[j] = b.in_slot(j); \\
    for (unsigned e = 0; e < 32; ++e) out[n + e] = b.has(e); \\
}
SLOTS(8) SLOTS(12) SLOTS(16) SLOTS(20)
extern "C" long shares(long heads, long T) { return l2kv::share_plan(heads, T, l2kv::kLongestShare); }
extern "C" int per_lane(long T) { return l2kv::score_keys_per_lane(T); }
extern "C" unsigned most(int per) { return l2kv::position_slots(per); }
extern "C" unsigned longest() { return l2kv::kLongestShare; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which(build.hipcc()) is None:
        pytest.skip("no hipcc")
    where = tmp_path_factory.mktemp("blocks")
    (where / "blocks.hip").write_text(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + build.CSRC, str(where / "blocks.hip"),
                    "-o", str(where / "blocks.so")], check=True, capture_output=True)
    lib = C.CDLL(str(where / "blocks.so"))
    lib.shares.argtypes, lib.shares.restype, lib.per_lane.argtypes = [C.c_long, C.c_long], C.c_long, [C.c_long]
    return lib


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


def test_a_share_fits_its_list_and_its_registers(lib):
    longest = lib.longest()
    edges = {k * 1024 + d for k in range(1, 33) for d in (0, 1, 1023)} | {longest, longest + 1, 2 * longest}
    for T in sorted(t for t in edges | set(range(1025, 32769, 61)) if 1024 < t <= 32768):
        blocks, slots = (T + 1023) // 1024, lib.most(lib.per_lane(T))
        for heads in (1, 2, 5, 16, 31, 32, 100, 128, 256, 257, 4000, 100000):
            shares = lib.shares(heads, T)
            assert 1 <= shares <= blocks <= shares * slots and (T + shares - 1) // shares <= longest, (T, heads)
