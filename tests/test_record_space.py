"""Copy records take workspace only for the levels that a plan records, on
the CPU build of the library."""
import ctypes as C

import numpy as np
import pytest

import gen


def _deep(orc, n=150_000, B=4096):
    x = gen.by_name("text", n, 41)
    a = orc.encode(x, block_size=B, interleave=16, min_match=8, hash_len=8, max_level=0, flags=2)
    assert orc.info(a)["depth"] >= 8
    return x, a


def test_plans_without_recorded_levels_reserve_no_records(orc):
    """A range of the first block has a plan of one level: its workspace holds
    the block's literals and bytes, and no records (139 KB a block here)."""
    import simt_lib
    B = 65536
    x, a = _deep(orc, 12 * B, B)
    one = np.array([0, 1000], dtype=np.uint64)
    assert simt_lib.Archive(a).workspace(one).size < 2 * B + 65536
    ooc = simt_lib.OocArchive(a)
    assert ooc.workspace_bytes(0, 1000) < 4 * B + 65536
    # the whole range's does: every block of its levels
    whole = simt_lib.Archive(a).workspace(np.array([0, len(x)], dtype=np.uint64)).size
    assert whole > 12 * (2 * B + 16 * (B // 8 + 512))
