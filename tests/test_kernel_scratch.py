"""No kernel of the library needs private memory: the runtime would have to find it for the queue at the first such launch, and
nothing here allocates."""
from paper_2406_11430_amd import binding

KEY = b".private_segment_fixed_size"


def test_no_private_memory():
    code = open(binding.LIB_PATH, "rb").read()
    sizes, at = [], code.find(KEY)
    while at >= 0:                                          # an unsigned number in the kernels' metadata (msgpack)
        at += len(KEY)
        lead = code[at]
        assert lead < 0x80 or lead in (0xcc, 0xcd, 0xce), lead
        sizes.append(lead if lead < 0x80 else int.from_bytes(code[at + 1:at + 1 + (1 << (lead - 0xcc))], "big"))
        at = code.find(KEY, at)
    assert len(sizes) > 100 and not any(sizes), sizes
