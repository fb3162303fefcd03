"""Match bytes whose sources straddle sequences, tiles or blocks: tiles with
few of them (followed one run at a time), with many (resolved in rounds) and
with several rounds, at every workgroup size, against the original bytes and
the oracle; the count of bytes read from earlier blocks with them."""
import numpy as np
import pytest

import gen


def _near(n, seed):
    """Copies from just behind, crossing the ends of what they copy, in long
    chains; now and then from far back."""
    rng = np.random.default_rng(seed)
    out = bytearray(rng.integers(0, 256, 300, dtype=np.uint8).tobytes())
    while len(out) < n:
        back = int(rng.integers(17, min(len(out), 120 if rng.random() < 0.9 else 20_000)))
        m = int(rng.integers(18, 400))
        at = len(out) - back
        for i in range(m):
            out.append(out[at + i])
        out += rng.integers(0, 256, int(rng.integers(1, 4)), dtype=np.uint8).tobytes()
    return bytes(out[:n])


# input, n, B, cap
CASES = [("near", 40_000, 16384, 0), ("near", 150_000, 65536, 3), ("tandem", 120_000, 4096, 0),
         ("near", 300_000, 1 << 18, 0), ("near", 20_000, 1000, 2)]


def _archive(orc, case):
    name, n, B, cap = case
    x = _near(n, 11) if name == "near" else gen.tandem(n, 12)
    return x, orc.encode(x, block_size=B, interleave=8, min_match=16, hash_len=16, max_level=cap, flags=2)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d-B%d-cap%d" % c)
def test_slow_bytes_cpu_build(orc, case):
    import simt_lib
    x, a = _archive(orc, case)
    arc = simt_lib.Archive(a)
    counts = []
    for waves in (1, 2, 8):
        got, ext = simt_lib.decode_all_ext(arc, dict(mode=1, waves_per_block=waves))
        assert got == x, waves
        counts.append(ext)
    lo, hi = len(x) // 3, len(x) - 7
    assert arc.seek_device(lo, hi) == x[lo:hi]  # blocks in slots: sources cross non-adjacent blocks
    assert (counts[0] > 0) == (arc.depth > 1)  # bytes from earlier blocks where there are levels


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES + [("near", 1_000_000, 16384, 4)], ids=lambda c: "%s-%d-B%d-cap%d" % c)
def test_slow_bytes_gpu(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive
    x, a = _archive(orc, case)
    want = np.frombuffer(x, np.uint8)
    arc = Archive(a, device="cuda:0")
    for tuning in [dict(mode=1, waves_per_block=w) for w in (0, 1, 2, 4, 8)] + [dict(mode=2)]:
        out = arc.decode_all(tuning=tuning)
        arc.check()
        assert np.array_equal(out.cpu().numpy(), want), tuning
    lo, hi = len(x) // 3, len(x) - 7
    for plan in ("host", "device"):
        got = arc.seek(lo, hi, plan=plan)
        arc.check()
        assert got.cpu().numpy().tobytes() == x[lo:hi], plan
