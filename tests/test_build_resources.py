"""Resources of the built kernels, read from the code objects' metadata in
the library: what the compiler reports, checked without a GPU."""
import re

import pytest

from paper_2205_14465_amd import binding as B


def _kernels():
    """{mangled name: bytes of scratch a lane} of every kernel in the library:
    the metadata's keys come in alphabetical order, so a kernel's name is
    followed by its private segment size (a msgpack integer)."""
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_Z[\w.]+?)\xbb\.private_segment_fixed_size(.)(....)",
                         data, re.S):
        tag, rest = m.group(2)[0], m.group(3)
        size = tag if tag < 0x80 else {0xcc: rest[0], 0xcd: int.from_bytes(rest[:2], "big"),
                                       0xce: int.from_bytes(rest, "big")}[tag]
        out[m.group(1).decode()] = size
    return out


@pytest.mark.parametrize("kernel", ["sign_onepass", "quant_onepass"])
def test_one_pass_kernels_use_no_scratch(kernel):
    """Chunks in flight live in registers: an array that the compiler moves
    to scratch makes the loads wait before the next chunk's go out."""
    found = {n: s for n, s in _kernels().items() if kernel + "I" in n}
    assert len(found) >= 3, sorted(_kernels())
    assert all(s == 0 for s in found.values()), found
