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
