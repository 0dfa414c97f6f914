"""The rule by which the work list of an ordered ragged batch cuts its sequences (csrc/ragged_plan.hpp), on the host."""
import ctypes as C
import random
import shutil
import subprocess

import pytest

from paper_2406_11430_amd import build

SOURCE = """
#include <hip/hip_runtime.h>
#include "ragged_plan.hpp"
extern "C" int pieces(long cus, int n_seq, int hkv, long slots, int most, int longest) {
    return l2kv::ragged_pieces(l2kv::ragged_rule(cus, n_seq, hkv, slots, most), longest);
}
"""


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    if shutil.which(build.hipcc()) is None:
        pytest.skip("no hipcc")
    where = tmp_path_factory.mktemp("plan")
    (where / "plan.hip").write_text(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + build.CSRC, str(where / "plan.hip"),
                    "-o", str(where / "plan.so")], check=True, capture_output=True)
    lib = C.CDLL(str(where / "plan.so"))
    lib.pieces.argtypes = [C.c_long, C.c_int, C.c_int, C.c_long, C.c_int, C.c_int]

    def of(lens, Hkv=8, most=8, cus=256):
        return lib.pieces(cus, len(lens), Hkv, sum(lens), most, max(lens))
    return of


@pytest.mark.parametrize("n,want", [(12, 2), (16, 2), (20, 1), (24, 1), (28, 1), (32, 1), (40, 1), (64, 1)])
def test_alike(pieces, n, want):
    assert pieces([4000] * n) == want
    assert pieces([4000 - 37 * (i % 9) for i in range(n)]) == want


@pytest.mark.parametrize("n", range(18, 33))
def test_one_long_sequence(pieces, n):
    """One more sequence does not make the launch wait for a piece twice as long."""
    lens = [8000] + [500] * (n - 1)
    load = sum(lens) * 8 / 256
    assert 5 <= pieces(lens) <= 8 and 8000 / pieces(lens) <= 2.5 * load
    assert abs(pieces(lens) - pieces(lens + [500])) <= 2


def test_few_long_sequences(pieces):
    assert pieces([8000] * 4 + [500] * 20) == 4 and pieces([8000] * 4 + [500] * 27) == 4
    assert pieces([8000] + [500] * 63) == 4 and pieces([8000] + [2000] * 30) == 3
    assert pieces([8000] + [500] * 15) == 8                           # already split for the compute units


def test_long_sequences_are_split_whatever_the_load(pieces):
    for rows, want in ((16384, 1), (16385, 2), (40000, 3), (70000, 5)):
        assert pieces([rows] * 200) == want
    assert pieces([300000] * 200) == 8 and pieces([300000] * 200, most=3) == 3


def test_any_numbers(pieces):
    rng = random.Random(1)
    for _ in range(3000):
        n = rng.choice([1, 2, 7, 60, 8191])
        hi = rng.choice([1, 64, 5000, 2 ** 31 // n - 1])
        lens = [rng.randint(0, hi) for _ in range(n - 1)] + [max(1, hi)]
        most = rng.randint(1, 8)
        assert 1 <= pieces(lens, Hkv=rng.choice([1, 3, 8]), most=most, cus=rng.choice([1, 32, 256, 304])) <= most
