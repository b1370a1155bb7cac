"""No kernel of the built library has a private segment (register spills, indexed local arrays).

A kernel with one needs scratch memory from the runtime at its first launch; when the allocation caches
hold the device's memory that allocation fails and the runtime ends the process, where a
failed hipMalloc of the library would give the caches back and go on.
"""
import os

import pytest

from paper_2207_04620_amd import he

KEY = b".private_segment_fixed_size"


def test_kernels_have_no_private_segment():
    if not os.path.exists(he.LIB_PATH):
        pytest.skip("libhe.so not built")
    data = open(he.LIB_PATH, "rb").read()
    at, n = data.find(KEY), 0
    while at >= 0:
        # the metadata is MessagePack: the key's value follows it, and 0 is the byte 0
        assert data[at + len(KEY)] == 0, f"kernel metadata at {at}: a private segment"
        n += 1
        at = data.find(KEY, at + 1)
    assert n >= 40, f"{n} kernels found"
