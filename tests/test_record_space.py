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


def _batch_sizes(arc, lib, cap, nb, B):
    """The size that the size function states, and what a context needed
    before it held records and the whole-archive plan's entries (8 bytes a
    block for the blocks' ids and counts instead)."""
    b = C.c_uint64(0)
    assert lib.ace_batch_workspace_bytes(arc, cap, C.byref(b)) == 0
    return b.value, b.value - nb * (64 + 16 * (B // 8 + 512)) + 8 * nb


@pytest.mark.parametrize("cap", [1, 5])
def test_batches_do_without_room_for_records_and_plan(orc, cap):
    import simt_lib
    L = simt_lib.lib()
    x, a = _deep(orc)
    arc = simt_lib.Archive(a)
    nb = arc.n_blocks
    need, bare = _batch_sizes(arc._h, L, cap, nb, 4096)
    rng = np.random.default_rng(3)
    lo = np.sort(rng.integers(0, len(x) - 9000, cap)).astype(np.uint64)
    hi = lo + rng.integers(1, 9000, cap).astype(np.uint64)
    want = [x[int(l):int(h)] for l, h in zip(lo, hi)]
    r = np.empty(2 * cap, dtype=np.uint64)
    r[0::2], r[1::2] = lo, hi
    ln = (hi - lo).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(ln)[:-1]]).astype(np.uint64)
    for size in (need, need - 1, bare):
        ws = np.zeros(size + 4096, dtype=np.uint8)
        ws[size:] = 0xA5
        h = C.c_void_p()
        assert L.ace_batch_create(arc._h, cap, simt_lib._p(ws), size, None, C.c_void_p(L.simt_stream_create()),
                                  C.byref(h)) == 0, size
        for _ in range(2):
            out = np.zeros(int(ln.sum()), dtype=np.uint8)
            assert L.ace_batch_run(h, simt_lib._p(r), cap, simt_lib._p(out), simt_lib._p(off)) == 0
            assert out.tobytes() == b"".join(want)
        assert L.ace_check(simt_lib._p(ws), None) == 0 and (ws[size:] == 0xA5).all()
        L.ace_batch_destroy(h)
    assert L.ace_batch_create(arc._h, cap, simt_lib._p(ws), bare // 2, None, C.c_void_p(L.simt_stream_create()),
                              C.byref(h)) == -4  # ACE_E_NOSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("name,n,B,W,mlv,flags", [("text", 150_000, 4096, 16, 0, 2), ("mixed", 3 << 20, 16384, 32, 8, 0)])
def test_bare_batches_gpu(orc, name, n, B, W, mlv, flags):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive, aceseek
    L = aceseek.lib()
    x = gen.by_name(name, n, 41)
    a = orc.encode(x, block_size=B, interleave=W, min_match=16, hash_len=16, max_level=mlv, flags=flags)
    arc = Archive(a, device="cuda:0")
    b = C.c_uint64(0)
    assert L.ace_batch_workspace_bytes(arc._h, 40, C.byref(b)) == 0
    bt = arc.batch(40)
    bt.close()
    ws = torch.zeros(b.value, dtype=torch.uint8, device="cuda:0")
    h = C.c_void_p()
    assert L.ace_batch_create(arc._h, 40, C.c_void_p(ws.data_ptr()), b.value - 1, None,
                              C.c_void_p(bt.stream.cuda_stream), C.byref(h)) == 0
    torch.cuda.synchronize()
    for seed in (1, 2, 3):
        lo, hi = gen.seek_requests(n, 40, seed, max_len=n // 3)
        ln = (hi - lo).astype(np.int64)
        off = np.concatenate([[0], np.cumsum(ln)[:-1]]).astype(np.uint64)
        r = np.empty(80, dtype=np.uint64)
        r[0::2], r[1::2] = lo, hi
        out = torch.zeros(int(ln.sum()), dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        assert L.ace_batch_run(h, r.ctypes.data_as(C.c_void_p), 40, C.c_void_p(out.data_ptr()),
                               off.ctypes.data_as(C.c_void_p)) == 0
        assert L.ace_check(C.c_void_p(ws.data_ptr()), C.c_void_p(bt.stream.cuda_stream)) == 0
        assert out.cpu().numpy().tobytes() == b"".join(x[int(l):int(k)] for l, k in zip(lo, hi))
    L.ace_batch_destroy(h)
