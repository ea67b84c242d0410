"""`-m gpu`: slots assigned from the list of victims (up to 4096 of them, no slot empty before) and by counting empty slots: one victim, counts
that are no whole vectors, all slots of a tile, caches of whole tiles and not, either side of the limit, a cold cache filling up before,
plain and planned calls, and batches after which the guess of how many there will be is wrong."""
import pytest

from tests.parity import run_parity, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cache,distinct", [(1_100_000, 1, 1), (1_100_000, 1023, 700), (1_100_000, 1024, 1024), (1_100_000, 3073, 2999),
                                                 (1_100_000, 4500, 4090), (1_100_000, 4500, 4200), (6000, 5000, 4990)])
@pytest.mark.parametrize("dma", [False, True])
@pytest.mark.parametrize("warm", [False, True])
def test_slots_from_the_victims(rows, cache, distinct, dma, warm):
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=cache, seed=cache + distinct, multi_hot=False, bags=max(1, 6 * distinct), distinct_cap=distinct)
    run_parity(w, 5, warm=warm, dma_evict=dma)
    run_parity_planned(w, 5, warm=warm, dma_evict=dma)


def test_more_victims_than_the_batch_before_had():
    class Uneven(TinyWorkload):
        def batch(self, t):
            ids, off = super().batch(t)
            return (ids, off) if t % 2 else (ids % 40, off)

    w = Uneven(num_rows=1_100_000, dim=8, cache_rows=20_000, seed=1, multi_hot=False, bags=60_000, distinct_cap=19_000)
    run_parity_planned(w, 8, warm=True, dma_evict=True)


@pytest.mark.parametrize("rows,cache,bags,counted", [(300_000, 100_000, 250_000, False), (500_000, 200_000, 250_000, True), (2_500_000, 2_000_000, 8192, False), (2_500_000, 2_000_000, 20_000, True)])
def test_a_wrong_guess_is_bounded(rows, cache, bags, counted):
    """Planned batches after one of few victims: the list is read by every slot tile only while that stays bounded if there should be as many
    victims as lookups or slots.  Either way the slots are the oracle's."""
    import numpy as np
    import torch
    from paper_2208_05321_amd import FreqCache
    few, many = 40, min(bags, cache) * 4 // 5

    class Shift(TinyWorkload):
        def batch(self, t):
            ids = np.arange(bags) % (min(bags, cache) - many)
            m, first = (many, cache + 10 * few) if t == 2 else (few, cache + t * few)
            ids[:m] = first + np.arange(m)
            return self.by_rank[ids].astype(np.int64), np.arange(bags + 1, dtype=np.int64)

    w = Shift(num_rows=rows, dim=4, cache_rows=cache, seed=7, multi_hot=False, bags=bags)
    w.by_rank = np.argsort(w.freq_rank)
    run_parity_planned(w, 4, warm=True, dma_evict=True)
    gpu = FreqCache(rows, 4, cache, w.freq_rank, dma_evict=True)
    gpu.host_weight()[:] = 0
    gpu.warm()
    for t in range(3):
        ids, off = (torch.from_numpy(x).cuda() for x in w.batch(t))
        gpu.check()
        gpu.profile(t > 0)
        gpu.prepare(ids, off) if t == 0 else gpu.plan_next(ids, off)
        gpu.advance()
    rep = gpu.profile_report()
    gpu.close()
    assert rep["free_assign"]["launches"] == 1 and ("free_count" in rep) == counted, rep
