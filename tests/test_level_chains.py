"""Runs of small dependency levels (archives without a level cap), copied
level after level from records made ahead: blocks of one tile and of several,
blocks whose records do not fit or that have too many tiles (expanded when
their turn comes), short-period matches, 8-byte offsets, blocks that end
the archive short; whole decodes, seeks planned on the host and on the device
and batches, against the original bytes."""
import numpy as np
import pytest

import gen

# corpus, n, B, min_match, flags
CASES = [
    ("genome", 200_000, 4096, 20, 2),        # one tile a block
    ("text", 150_000, 16384, 4, 2),          # more records than there is room for
    ("text", 700_000, 1 << 17, 5, 2),        # more tiles than are recorded
    ("text", 400_001, 65536, 16, 6),         # several tiles, 8-byte offsets, short last block
    ("tandem", 120_000, 3000, 16, 0),        # short periods
    ("text", 30_000, 100, 8, 2),             # blocks of a few pieces, hundreds of levels
]


def _archive(orc, case):
    name, n, B, mm, flags = case
    x = gen.by_name(name, n, 41)
    a = orc.encode(x, block_size=B, interleave=16, min_match=mm, hash_len=mm, max_level=0, flags=flags)
    assert orc.info(a)["depth"] >= 4
    return x, a


def _id(c):
    return "%s-n%d-B%d-mm%d-f%d" % c


@pytest.mark.parametrize("case", [c for c in CASES if c[1] < 500_000], ids=_id)
def test_chains_cpu_build(orc, case):
    import simt_lib
    x, a = _archive(orc, case)
    arc = simt_lib.Archive(a)
    got, ext = simt_lib.decode_all_ext(arc, None)
    assert got == x
    # the same bytes are counted as from earlier blocks with a launch per level
    if case[1] // case[2] < 64:
        assert simt_lib.decode_all_ext(arc, dict(mode=1, waves_per_block=8)) == (x, ext)
    lo, hi = len(x) // 2 + 3, len(x) - 5
    assert arc.seek(lo, hi) == x[lo:hi]
    assert arc.seek_device(lo, hi) == x[lo:hi]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES + [("genome", 6 << 20, 4096, 20, 0)], ids=_id)
def test_chains_gpu(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive, OutOfCoreArchive
    x, a = _archive(orc, case)
    want = np.frombuffer(x, np.uint8)
    for resident in (True, False):
        arc = Archive(a, device="cuda:0", resident_plan=resident)
        ext = []
        for tuning in (None, None, dict(mode=1, waves_per_block=8)):
            out = torch.zeros(len(x), dtype=torch.uint8, device="cuda:0")
            arc.decode_all(out=out, tuning=tuning)
            arc.check()
            assert np.array_equal(out.cpu().numpy(), want), tuning
            ext.append(arc.read_counters()["ext_src_bytes"])
        assert ext[0] == ext[1]
        if case[3] >= 16:  # one tile a block at either size: the same count
            assert ext[0] == ext[2] or case[2] > 16384
    arc = Archive(a, device="cuda:0")
    ooc = OutOfCoreArchive(a, device="cuda:0")
    lo, hi = gen.seek_requests(len(x), 6, 3, max_len=len(x) // 2)
    for l, h in [(int(l), int(h)) for l, h in zip(lo, hi)] + [(len(x) - 1, len(x))]:
        for plan in ("host", "device"):
            got = arc.seek(l, h, plan=plan)
            arc.check()
            assert got.cpu().numpy().tobytes() == x[l:h], plan
        got = ooc.seek(l, h)
        ooc.check()
        assert got.cpu().numpy().tobytes() == x[l:h]
    bt = arc.batch(6)
    out = torch.zeros(int((hi - lo).sum()), dtype=torch.uint8, device="cuda:0")
    for _ in range(3):
        out.zero_()
        bt.run((lo, hi), out)
        bt.check()
        assert out.cpu().numpy().tobytes() == b"".join(x[int(l):int(h)] for l, h in zip(lo, hi))


# corpus, n, B, cap: groups of levels copied by a launch each; the last has
# levels inside and outside the recorded groups
GROUPS = [("text", 160_000, 200, 5), ("fastq", 1_500_000, 2000, 16), ("mixed", 4 << 20, 1000, 6)]


def _capped(orc, case):
    name, n, B, cap = case
    x = gen.by_name(name, n, 43)
    return x, orc.encode(x, block_size=B, interleave=16, min_match=16, hash_len=16, max_level=cap, flags=2)


@pytest.mark.parametrize("case", GROUPS[:1], ids=lambda c: "%s-n%d-B%d-cap%d" % c)
def test_recorded_groups_cpu_build(orc, case):
    import simt_lib
    x, a = _capped(orc, case)
    arc = simt_lib.Archive(a)
    assert arc.depth >= 3
    assert arc.decode_all() == x
    lo, hi = len(x) // 2 + 3, len(x) - 5
    assert arc.seek(lo, hi) == x[lo:hi]
    assert arc.seek_device(lo, hi) == x[lo:hi]


@pytest.mark.gpu
@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "%s-n%d-B%d-cap%d" % c)
def test_recorded_groups_gpu(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive
    x, a = _capped(orc, case)
    for resident in (True, False):
        arc = Archive(a, device="cuda:0", resident_plan=resident)
        out = torch.zeros(len(x), dtype=torch.uint8, device="cuda:0")
        arc.decode_all(out=out)
        arc.check()
        assert np.array_equal(out.cpu().numpy(), np.frombuffer(x, np.uint8))
    arc = Archive(a, device="cuda:0")
    lo, hi = gen.seek_requests(len(x), 5, 3, max_len=len(x))
    for l, h in [(int(l), int(h)) for l, h in zip(lo, hi)] + [(0, len(x)), (len(x) - 1, len(x))]:
        for plan in ("host", "device"):
            got = arc.seek(l, h, plan=plan)
            arc.check()
            assert got.cpu().numpy().tobytes() == x[l:h], plan
