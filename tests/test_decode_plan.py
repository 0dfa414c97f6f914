"""The plan of uniform decode launches (csrc/decode_plan.hip), on the host: what every plan has to hold to, over all head counts."""
import ctypes as C
import shutil
import subprocess

import pytest

from paper_2406_11430_amd import build

SOURCE = """
#include "decode_plan.hip"
namespace l2kv { int device_compute_units() { return 256; } }
extern "C" int splits(int heads, int group, long rows, int D, int bytes) {
    return l2kv::decode_plan(1, heads, group, rows, D, bytes, 0).n_splits;
}
extern "C" long scratch(int heads, int group, int n_splits, int D) { return (long)l2kv::decode_scratch_bytes(1, heads, group, n_splits, D); }
extern "C" long limit() { return L2KV_STATIC_SCRATCH_BYTES; }
extern "C" int work_list(int n_seq, int hkv, long rows, int n_splits) { return l2kv::decode_plan_ragged(n_seq, hkv, rows, rows, n_splits, true).worklist_wgs; }
extern "C" int max_splits(long rows) { return l2kv::decode_max_splits(rows); }
"""
ROWS = [(128, 2, 8), (64, 2, 8), (256, 2, 4), (128, 4, 8), (64, 4, 8)]    # elements, bytes each, largest group
LENGTHS = [1, 64, 65, 200, 256, 257, 700, 1024, 1500, 2048, 2600, 3072, 4096, 5120, 8192, 8193, 20000, 40000, 131072]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which(build.hipcc()) is None:
        pytest.skip("no hipcc")
    where = tmp_path_factory.mktemp("decode_plan")
    (where / "plan.hip").write_text(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + build.CSRC, str(where / "plan.hip"),
                    "-o", str(where / "plan.so")], check=True, capture_output=True)
    lib = C.CDLL(str(where / "plan.so"))
    lib.splits.argtypes = [C.c_int, C.c_int, C.c_long, C.c_int, C.c_int]
    lib.scratch.argtypes, lib.scratch.restype = [C.c_int] * 4, C.c_long
    lib.limit.restype = C.c_long
    lib.max_splits.argtypes = [C.c_long]
    lib.work_list.argtypes = [C.c_int, C.c_int, C.c_long, C.c_int]
    return lib


@pytest.mark.parametrize("D,bytes,most", ROWS)
def test_without_a_workspace(lib, D, bytes, most):
    """l2kv_decode_attn_static takes the plan of l2kv_decode_attn, whose partial results have to fit its scratch memory wherever those of
    one workgroup for each head do."""
    limit = lib.limit()
    for group in range(1, most + 1):
        for rows in LENGTHS:
            for heads in range(1, 1201):
                n = lib.splits(heads, group, rows, D, bytes)
                assert 1 <= n <= lib.max_splits(rows)
                assert lib.scratch(heads, group, n, D) <= limit or lib.scratch(heads, group, 1, D) > limit, (heads, group, rows, n)


@pytest.mark.parametrize("heads,group,rows,D,bytes,n", [
    (80, 3, 256, 128, 2, 2), (80, 3, 257, 128, 2, 3), (56, 1, 384, 128, 2, 3), (56, 1, 385, 128, 2, 4), (56, 4, 576, 128, 4, 3)])
def test_one_more_split_shortens_the_longest(lib, heads, group, rows, D, bytes, n):
    assert lib.splits(heads, group, rows, D, bytes) == n


@pytest.mark.parametrize("heads,group,rows,D,bytes,n", [
    (4, 2, 2048, 256, 2, 32), (4, 2, 2049, 256, 2, 17), (4, 2, 2826, 256, 2, 23), (3, 4, 2826, 256, 2, 23), (2, 2, 2826, 256, 2, 45), (4, 2, 2826, 128, 4, 45)])
def test_streams_behind_two_round_trips(lib, heads, group, rows, D, bytes, n):
    assert lib.splits(heads, group, rows, D, bytes) == n


@pytest.mark.parametrize("heads,group,rows,D,bytes,n", [
    (544, 8, 4096, 128, 2, 1), (513, 6, 2600, 128, 2, 1), (513, 3, 1500, 256, 2, 1), (576, 5, 4096, 128, 2, 1), (529, 5, 4096, 128, 2, 3),
    (530, 5, 4096, 128, 2, 1), (330, 8, 2048, 128, 2, 3), (331, 8, 2048, 128, 2, 1), (597, 4, 4096, 128, 2, 3)])
def test_three_where_they_fit(lib, heads, group, rows, D, bytes, n):
    assert lib.splits(heads, group, rows, D, bytes) == n


def test_a_work_list_has_no_more_items_than_its_counter_counts(lib):
    assert lib.work_list(16384, 1, 20000, 255) == 256 and lib.work_list(2048, 8, 20000, 256) == 0
    assert lib.work_list(65535, 1, 20000, 63) == 256 and lib.work_list(65535, 1, 20000, 65) == 0 and lib.work_list(65535, 1, 20000, 0) == 256
