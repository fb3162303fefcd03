"""Device-side planning at the edges of its compaction chunks (1,024 blocks;
up to eight chunks in one launch, more in three): single seeks and a replayed
batch, against the original bytes."""
import numpy as np
import pytest

import gen

BLOCKS = [1, 1023, 1024, 1025, 8192, 8193]
B = 24


def _archive(orc, nb):
    n = nb * B - 5
    x = gen.text(n, 17)
    a = orc.encode(x, block_size=B, interleave=4, min_match=6, hash_len=6, max_level=5, flags=2)
    assert orc.info(a)["n_blocks"] == nb
    rng = np.random.default_rng(nb)
    lo = np.sort(rng.integers(0, n, 6)).astype(np.uint64)
    hi = np.minimum(lo + rng.integers(1, 3000, 6).astype(np.uint64), n).astype(np.uint64)
    lo[0], hi[5] = 0, n
    return x, a, lo, hi


@pytest.mark.parametrize("nb", BLOCKS)
def test_planner_cpu_build(orc, nb):
    import simt_lib
    x, a, lo, hi = _archive(orc, nb)
    arc = simt_lib.Archive(a)
    for l, h in [(int(lo[0]), int(hi[0])), (int(lo[5]), int(hi[5]))]:
        assert arc.seek_device(l, h) == x[l:h], (l, h)
    got = simt_lib.seek_batch_graph(arc, lo[:3], hi[:3])
    assert all(g == x[int(l):int(h)] for g, l, h in zip(got, lo, hi))


@pytest.mark.gpu
@pytest.mark.parametrize("nb", BLOCKS)
def test_planner_gpu(orc, nb):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive
    x, a, lo, hi = _archive(orc, nb)
    arc = Archive(a, device="cuda:0")
    ws = torch.zeros(arc.seek_device_bytes(), dtype=torch.uint8, device="cuda:0")
    for l, h in zip(lo.tolist(), hi.tolist()):
        for plan in ("device", "auto", "host"):
            got = arc.seek(l, h, ws=ws, plan=plan)
            arc.check(ws)
            assert got.cpu().numpy().tobytes() == x[l:h], (l, h, plan)
    bt = arc.batch(6)
    out = torch.zeros(int((hi - lo).sum()), dtype=torch.uint8, device="cuda:0")
    # runs one after another without a wait between: the second's descriptors
    # are staged while the first may still run
    for k in (0, 3, 0):
        bt.run((lo[k:], hi[k:]), out)
    bt.check()
    assert out.cpu().numpy().tobytes() == b"".join(x[l:h] for l, h in zip(lo.tolist(), hi.tolist()))
