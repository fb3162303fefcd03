"""Workspaces whose first 256 bytes are zero and whose other bytes hold
anything, as the header asks: every entry point gives the original bytes, on
the CPU build and through the binding's own workspaces."""
import ctypes as C

import numpy as np
import pytest

import gen

# corpus, n, B, cap
CASES = [("text", 60_000, 2000, 0), ("text", 160_000, 200, 5)]


def _archive(orc, case, flags=0):
    name, n, B, cap = case
    x = gen.by_name(name, n, 41)
    return x, orc.encode(x, block_size=B, interleave=16, min_match=8, hash_len=8, max_level=cap, flags=flags)


def _id(c):
    return "%s-n%d-B%d-cap%d" % c


def _dirty(n):
    ws = np.full(max(n, 256), 0xA5, dtype=np.uint8)
    ws[:256] = 0
    return ws


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_dirty_workspaces_cpu_build(orc, case):
    import simt_lib
    L, p = simt_lib.lib(), simt_lib._p
    x, a = _archive(orc, case)
    arc = simt_lib.Archive(a)
    n = len(x)
    lo, hi = n // 3, n - 77
    for mode in (0, 2) if case[3] == 0 else (0,):
        t = simt_lib.Tuning(mode=mode)
        ws = _dirty(arc.workspace().size)
        out = np.zeros(n, dtype=np.uint8)
        assert L.ace_decode_all(arc._h, p(out), n, p(ws), ws.size, C.byref(t), None) == 0
        assert L.ace_check(p(ws), None) == 0 and out.tobytes() == x, mode
    r = np.array([lo, hi], dtype=np.uint64)
    ws = _dirty(arc.workspace(r).size)
    out = np.zeros(hi - lo, dtype=np.uint8)
    assert L.ace_seek(arc._h, lo, hi, p(out), p(ws), ws.size, None, None) == 0
    assert L.ace_check(p(ws), None) == 0 and out.tobytes() == x[lo:hi]
    b = C.c_uint64(0)
    assert L.ace_plan_bytes(arc._h, C.byref(b)) == 0
    plan = np.full(b.value, 0xA5, dtype=np.uint8)
    assert L.ace_archive_attach_plan(arc._h, p(plan), b.value, None) == 0
    assert L.ace_batch_workspace_bytes(arc._h, 1, C.byref(b)) == 0
    ws = _dirty(b.value)
    out[:] = 0
    assert L.ace_seek(arc._h, lo, hi, p(out), p(ws), ws.size, None, None) == 0
    assert L.ace_check(p(ws), None) == 0 and out.tobytes() == x[lo:hi]
    ws, off, h = _dirty(b.value), np.zeros(1, dtype=np.uint64), C.c_void_p()
    assert L.ace_batch_create(arc._h, 1, p(ws), ws.size, None, C.c_void_p(L.simt_stream_create()), C.byref(h)) == 0
    for _ in range(2):
        out[:] = 0
        assert L.ace_batch_run(h, p(r), 1, p(out), p(off)) == 0
        assert out.tobytes() == x[lo:hi]
    L.ace_batch_destroy(h)
    ooc = simt_lib.OocArchive(a)
    ws = _dirty(ooc.workspace_bytes(lo, hi))
    out[:] = 0
    assert L.ace_seek_ooc(ooc._h, lo, hi, p(out), p(ws), ws.size, None, None) == 0
    assert L.ace_check(p(ws), None) == 0 and out.tobytes() == x[lo:hi]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES + [("mixed", 3 << 20, 16384, 0), ("mixed", 6 << 20, 4096, 8)], ids=_id)
def test_dirty_workspaces_gpu(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive, OutOfCoreArchive
    x, a = _archive(orc, case)
    n = len(x)
    lo, hi = n // 3, n - 77

    def dirty(size):
        ws = torch.full((max(size, 256),), 0xA5, dtype=torch.uint8, device="cuda:0")
        ws[:256] = 0
        return ws

    def same(t, want, ws, arc):
        arc.check(ws)
        assert t.cpu().numpy().tobytes() == want

    arc = Archive(a, device="cuda:0")
    for mode in (0, 2, 3):
        ws = dirty(arc.workspace_bytes())
        same(arc.decode_all(ws=ws, tuning=dict(mode=mode)), x, ws, arc)
    ws = dirty(arc.workspace_bytes([lo, hi]))
    same(arc.seek(lo, hi, ws=ws, plan="host"), x[lo:hi], ws, arc)
    ws = dirty(arc.seek_device_bytes())
    same(arc.seek(lo, hi, ws=ws, plan="device"), x[lo:hi], ws, arc)
    r = [lo, hi, 5, 900]
    ws = dirty(arc.workspace_bytes(r))
    same(arc.seek_batch(r, ws=ws), x[lo:hi] + x[5:900], ws, arc)
    ooc = OutOfCoreArchive(a, device="cuda:0")
    ws = dirty(ooc.workspace_bytes(lo, hi))
    same(ooc.seek(lo, hi, ws=ws), x[lo:hi], ws, ooc)
    # the binding's own workspaces, where memory was used before
    del ws, arc, ooc
    torch.cuda.synchronize()
    junk = torch.full((256 << 20,), 0xA5, dtype=torch.uint8, device="cuda:0")
    del junk
    arc, ooc = Archive(a, device="cuda:0"), OutOfCoreArchive(a, device="cuda:0")
    same(arc.seek(lo, hi), x[lo:hi], None, arc)
    same(arc.decode_all(), x, None, arc)
    same(arc.seek_batch(r), x[lo:hi] + x[5:900], None, arc)
    same(ooc.seek(lo, hi), x[lo:hi], None, ooc)
