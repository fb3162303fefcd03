"""The gather of decoded ranges, split over several workgroups per request:
ranges that start and end inside 16-byte chunks, cross many block edges
(blocks shorter than a chunk among them), and need more steps than the
launch has workgroups per request."""
import numpy as np
import pytest

import gen

# n, B, ranges: below one step, at its edges, several steps
SHAPES = [
    (60_000, 37, [(0, 1), (36, 38), (5, 16384 + 5), (17, 59_999)]),
    (90_001, 1000, [(999, 17_384), (1, 16_385), (3, 90_001), (90_000, 90_001)]),
    (200_003, 16384, [(16_383, 32_769), (1, 200_002), (0, 200_003), (15, 31)]),
]


@pytest.mark.parametrize("n,B,ranges", SHAPES)
def test_gather_edges_cpu_build(orc, n, B, ranges):
    import simt_lib
    x = gen.by_name("text", n, 3)
    a = orc.encode(x, block_size=B, interleave=8, min_match=16, hash_len=16, max_level=4)
    arc = simt_lib.Archive(a)
    for lo, hi in ranges:
        assert arc.seek_device(lo, hi) == x[lo:hi], (lo, hi)
    lo, hi = np.array(ranges, dtype=np.uint64).T
    got = simt_lib.seek_batch_graph(arc, lo, hi)
    assert all(g == x[int(l):int(h)] for g, l, h in zip(got, lo, hi))


@pytest.mark.gpu
@pytest.mark.parametrize("cap", [1, 3, 8192])
def test_gather_more_steps_than_workgroups(cap):
    """Requests longer than the launch's workgroups cover in one step each
    (capacity 8192: one workgroup per request)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive, encode
    n = (18 << 20) + 11
    x = gen.random_bytes(n, 9)
    arc = Archive(encode(x, max_level=4), device="cuda:0")
    bt = arc.batch(cap)
    ranges = [(3, n - 2), (7, 40_001), (16_383, 16_385)][:min(cap, 3)]
    lo, hi = np.array(ranges, dtype=np.uint64).T
    out = torch.zeros(int((hi - lo).sum()), dtype=torch.uint8, device="cuda:0")
    bt.run((lo, hi), out)
    bt.check()
    assert out.cpu().numpy().tobytes() == b"".join(x[l:h] for l, h in ranges)
    got = arc.seek(5, n - 4, plan="device")
    arc.check()
    assert got.cpu().numpy().tobytes() == x[5:n - 4]
