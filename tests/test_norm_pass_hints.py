"""The cache hints of the norm pass in the code that the compiler makes: the pass over more keys than the caches hold
must store its results with the non-temporal hint (2 to 4 % of its time), and two stores that
differ in nothing else are easily merged into one without it, which no result shows."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_11430_amd import build

KERNELS = ["norms_kernelINS_3F32ELi64E", "norms_kernelINS_3F32ELi128E", "norms_kernelINS_4BF16ELi128E",
           "norms_kernelINS_4BF16ELi256E", "norms_row_pairs_kernelI"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which(build.hipcc()) is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "norms.s")
    subprocess.run([build.hipcc(), *build.HIPCC_FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "norms.hip"),
                    "-o", out], check=True, capture_output=True)
    bodies = {}
    name = None
    for line in open(out):
        label = re.match(r"(_ZN\S+):", line)
        if label:
            name = label.group(1)
            bodies[name] = []
        elif name:
            bodies[name].append(line)
            if "s_endpgm" in line:
                name = None
    return bodies


# caching: 0 = rows and results streamed, 1 = rows only, 2 = rows only up to the cached tail
@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("caching", [0, 1, 2])
def test_hints(assembly, kernel, caching):
    found = [b for n, b in assembly.items() if kernel in n and "NormCachingE%dE" % caching in n]
    assert len(found) == 1, [n for n in assembly if kernel in n]
    loads = [x for x in found[0] if re.search(r"\b(global|buffer)_load_dwordx4\b", x)]
    stores = [x for x in found[0] if re.search(r"\bglobal_store_dword\b", x)]
    streamed = [bool(re.search(r"\bnt\b", x)) for x in loads]
    assert loads and stores
    assert all(streamed) if caching < 2 else any(streamed) and not all(streamed)
    assert all(bool(re.search(r"\bnt\b", x)) == (caching == 0) for x in stores)
