"""The entropy decode's two table layouts (one word per slot in launches of up
to 2,304 blocks, a symbol map and one word per symbol above) at interleaves
that fill, repeat over or leave over the lanes of a wavefront, with every
stream rANS-coded, one-symbol streams among them."""
import numpy as np
import pytest

import gen

# n, B, W: blocks below and above the limit
SHAPES = [(24_000, 300, w) for w in (1, 5, 31, 32, 33, 63, 64)] + [(160_000, 64, w) for w in (3, 32, 40, 64)]


def _input(n):
    """Text, then one repeated byte (single-symbol streams), then all 256
    symbols (the largest table)."""
    return gen.text(n - n // 4 - n // 8, 5) + b"a" * (n // 8) + gen.random_bytes(n // 4, 6)


def _archive(orc, n, B, W):
    x = _input(n)
    a = orc.encode(x, block_size=B, interleave=W, min_match=16, hash_len=16, max_level=3, flags=1)
    assert (orc.info(a)["n_blocks"] > 2304) == (n == 160_000)
    return x, a


@pytest.mark.parametrize("n,B,W", [s for s in SHAPES if s[0] == 24_000] + [(160_000, 64, 40)])
def test_tables_cpu_build(orc, n, B, W):
    import simt_lib
    x, a = _archive(orc, n, B, W)
    assert simt_lib.Archive(a).decode_all(dict(mode=1)) == x


@pytest.mark.gpu
@pytest.mark.parametrize("n,B,W", SHAPES + [(300_000, 100_000, 64), (300_000, 100_000, 32)])
def test_tables_gpu(orc, n, B, W):
    """Also long streams, whose word ring wraps many times."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive
    x, a = _archive(orc, n, B, W)
    arc = Archive(a, device="cuda:0")
    for per_wave in (0, 1):
        out = arc.decode_all(tuning=dict(mode=1, blocks_per_wg=per_wave))
        arc.check()
        got = out.cpu().numpy()
        assert np.array_equal(got, np.frombuffer(x, np.uint8)), (per_wave, np.nonzero(got != np.frombuffer(x, np.uint8))[0][:4])
