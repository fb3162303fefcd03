"""A whole-archive decode without the resident plan copies its plan and its
level boundaries from pinned memory that the handle keeps: the call does not
wait for its stream, and a captured decode reads nothing that may be freed."""
import ctypes as C

import pytest

import gen


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_decode_copies_from_kept_pinned_memory(orc, mode):
    import simt_lib
    x = gen.by_name("text", 30_000, 41)
    a = orc.encode(x, block_size=500, interleave=16, min_match=8, hash_len=8, max_level=0, flags=2)
    assert orc.info(a)["depth"] >= 4  # recorded groups of levels
    arc = simt_lib.Archive(a)
    count = simt_lib.lib().simt_pageable_copies
    count.restype = C.c_uint64
    count()
    assert arc.decode_all(dict(mode=mode)) == x
    assert count() == 0
