"""What the built library says of its force kernels' registers: none may keep
spilled registers for code that its lists do not reach."""
import os
import re
import struct

import msgpack
import pytest

from paper_1812_07313_amd import bhq, build


def _kernels():
    """The kernels' entries in the metadata notes of the library's device code."""
    bhq.lib()  # builds it where nothing is built
    with open(build.LIB, "rb") as f:
        d = f.read()
    out, name = {}, b"AMDGPU\0\0"
    at = d.find(name)
    while at >= 0:
        namesz, size, kind = struct.unpack("<III", d[at - 12:at])
        if (namesz, kind) == (7, 32):
            for k in msgpack.unpackb(d[at + 8:at + 8 + size])["amdhsa.kernels"]:
                out[k[".name"]] = k
        at = d.find(name, at + 1)
    return out


@pytest.mark.parametrize("kind", [2, 3], ids=["split_quad", "split_mono"])
def test_fp64_split_kernels_do_not_spill(kind):
    """The FP64 split kernels with a block per group (every shape) keep no
    registers in scratch memory, which each block would write again: what they
    did keep there was for cutoffs past their table, and cost lists of small
    groups half their time.  (The persistent kernels, whose few blocks stay,
    are not held to this.)"""
    ks = {n: k for n, k in _kernels().items() if re.search(r"force_kernelIdLi%dE" % kind, n)}
    assert len(ks) >= 8
    for n, k in ks.items():
        assert k[".private_segment_fixed_size"] == 0, n
        assert k[".vgpr_spill_count"] == 0, n
