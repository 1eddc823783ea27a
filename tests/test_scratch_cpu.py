"""No kernel of the library spills to scratch memory (no GPU).

A kernel with a private segment makes every hardware queue allocate scratch at
its first launch there, which the first call on a new stream then waits for. The
segment's size stands in each kernel's metadata in the built library.
"""
import re

import pytest


@pytest.fixture(scope="module")
def library():
    import os
    from paper_2403_15913_amd import kkt as K
    if not os.path.exists(K.LIB_PATH):
        from paper_2403_15913_amd import build
        build.build()
    with open(K.LIB_PATH, "rb") as fh:
        return fh.read()


def test_no_kernel_uses_scratch(library):
    # MessagePack: keys in order, a kernel's name before its segment's size (one byte up to 127, else a marker >= 0xcc)
    found = re.findall(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_ZN3kkt\w+?)\xbb\.private_segment_fixed_size(.)", library,
                       re.S)
    names = {n.decode() for n, _ in found}
    assert len(names) >= 40 and any("k_fwd" in n for n in names) and any("k_factor" in n for n in names)
    assert not [n.decode() for n, size in found if size != b"\x00"]
