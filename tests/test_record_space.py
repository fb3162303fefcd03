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


def _guarded(call, cap, out_len):
    """call(out, ws, cap) with a workspace of cap bytes and a guard behind
    it: the return code and the output."""
    import simt_lib
    L = simt_lib.lib()
    ws = np.zeros(cap + 4096, dtype=np.uint8)
    ws[cap:] = 0xA5
    out = np.zeros(max(out_len, 1), dtype=np.uint8)
    rc = call(L, simt_lib._p(out), simt_lib._p(ws), cap)
    assert (ws[cap:] == 0xA5).all()
    if rc == 0:
        assert L.ace_check(simt_lib._p(ws), None) == 0
    return rc, out[:out_len].tobytes()


@pytest.mark.parametrize("entry", ["seek", "batch", "ooc"])
def test_seeks_do_without_room_for_records(orc, entry):
    """A workspace that holds everything but the records (whose size the size
    functions include) is taken, and gives the same bytes."""
    import simt_lib
    x, a = _deep(orc)
    lo, hi = len(x) // 3, len(x) - 77
    r = np.array([lo, hi], dtype=np.uint64)
    off = np.zeros(1, dtype=np.uint64)
    if entry == "ooc":
        arc = simt_lib.OocArchive(a)
        need = arc.workspace_bytes(lo, hi)
    else:
        arc = simt_lib.Archive(a)
        need = arc.workspace(r).size

    def call(L, out, ws, cap):
        if entry == "seek":
            return L.ace_seek(arc._h, lo, hi, out, ws, cap, None, None)
        if entry == "ooc":
            return L.ace_seek_ooc(arc._h, lo, hi, out, ws, cap, None, None)
        return L.ace_seek_batch(arc._h, simt_lib._p(r), 1, out, simt_lib._p(off), ws, cap, None, None)

    # the blocks' records: 16 bytes for each of B / 8 + 512 of them
    bare = need - 36 * 16 * (4096 // 8 + 512)
    assert bare > 0
    for cap in (need, need - 1, bare):
        rc, got = _guarded(call, cap, hi - lo)
        assert rc == 0 and got == x[lo:hi], cap
    rc, _ = _guarded(call, 4096, hi - lo)
    assert rc == -4  # ACE_E_NOSPACE
