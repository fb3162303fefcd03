"""The host encoder's hash chains, linked by a pass per thread (below four
threads) or sorted by bucket range first: the same archive as the oracle's
from any number of threads, around the sizes where slices and bucket ranges
become more than one, with and without a level cap."""
import pytest

import gen

SIZES = [0, 7, 8, 9, 3000, 40_000, 70_000, 131_071, 131_073, 600_001]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("cap", [0, 3])
def test_chains_same_for_any_thread_count(orc, n, cap):
    from paper_2606_24531_amd import encode
    x = gen.tandem(n, 5) if n else b""
    kw = dict(block_size=1000, interleave=8, min_match=9, hash_len=8, max_chain=16, max_level=cap)
    want = orc.encode(x, **kw)
    for threads in (1, 3, 4, 13):
        assert encode(x, n_threads=threads, **kw) == want, threads
