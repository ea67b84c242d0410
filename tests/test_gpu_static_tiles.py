"""`-m gpu`: counting at the edges of its two tile sizes (4096 ids a workgroup up to 2^17 ids, 8192 beyond), the largest count of arrays
with 0 to 3 counters beyond whole vectors, and ranks where nearly all counts are alike or all differ, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4095, 4097, 1 << 17, (1 << 17) + 1, 200_003])
@pytest.mark.parametrize("rows", [1, 6, 4099, 1_000_000, 1_000_005])
@pytest.mark.parametrize("skewed", [True, False])
def test_counts_and_ranks(n, rows, skewed):
    import torch
    from paper_2208_05321_amd import FreqCounter
    rng = np.random.default_rng(n + rows)
    ids = np.minimum((rng.random(n) ** (8 if skewed else 1) * rows).astype(np.int64), rows - 1)
    ids[-1] = rows - 1                                     # the last counter, too
    f = FreqCounter(rows)
    f.add(torch.from_numpy(ids).cuda())
    rank, inv, counts = f.build(with_counts=True)
    f.close()
    want = np.bincount(ids, minlength=rows)
    order = np.argsort(-want, kind="stable")
    assert np.array_equal(counts, want) and np.array_equal(inv, order)
    assert np.array_equal(rank[order], np.arange(rows))


def test_builds_of_one_pass():
    """Counts of 11 bits on either side of 32 tiles: ranked in one pass on both, so that 65,536 rows do not take longer than 65,537."""
    import time
    import torch
    from paper_2208_05321_amd import FreqCounter
    best = {}
    for rows in (65_537, 65_536):
        ids = (rows ** np.random.default_rng(5).random(20_000)).astype(np.int64) - 1
        fc = FreqCounter(rows)
        fc.add(torch.from_numpy(ids).cuda())
        fr, inv, cnt = fc.build(with_counts=True)
        want = np.bincount(ids, minlength=rows)
        assert 1024 <= want.max() < 2048 and np.array_equal(cnt, want)
        assert np.array_equal(inv, np.argsort(-want, kind="stable")) and np.array_equal(fr[inv], np.arange(rows))
        times = []
        for _ in range(60):
            a = time.perf_counter()
            fc.build(with_counts=True)
            times.append(time.perf_counter() - a)
        best[rows] = min(times)
        fc.close()
    assert best[65_536] < 1.08 * best[65_537], best
