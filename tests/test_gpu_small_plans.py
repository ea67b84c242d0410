"""`-m gpu`: planned batches with few rows to move: fetched on the index stream up to 1.5 MB (with the sort in the same launch up to
10240 lookups), their victims stored into the landing block by the gather up to the same size (plain calls: 256 KB).  Sizes on
either side of each border, blocks with and without room for the ranks behind the rows, both ways to run ahead."""
import numpy as np
import pytest

from tests.parity import run_parity, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu

LIMIT, PLAIN_LIMIT = 3 << 19, 1 << 18


@pytest.mark.parametrize("bags", [700, 10_240, 10_241, 30_000])
@pytest.mark.parametrize("dim,distinct", [(5, 650), (128, LIMIT // 512 - 130), (128, LIMIT // 512 + 260), (130, PLAIN_LIMIT // 520 - 40), (130, PLAIN_LIMIT // 520 + 40)])
@pytest.mark.parametrize("staging", [0, 300])
def test_few_rows_to_move(bags, dim, distinct, staging):
    w = TinyWorkload(num_rows=20 * distinct, dim=dim, cache_rows=distinct + 50, seed=bags + dim, multi_hot=False, bags=bags, distinct_cap=distinct)
    run_parity_planned(w, 6, warm=True, dma_evict=True, inputs_ready=bags == 10_240, staging_rows=staging)
    run_parity(w, 5, warm=True, dma_evict=True, staging_rows=staging, values_every=4)


@pytest.mark.parametrize("bags,dim,many,staging,inputs_ready,dirty", [
    (9000, 128, 2 * LIMIT // 512, 0, False, False), (9000, 128, 2 * LIMIT // 512 + 1, 0, True, False), (30_000, 128, 2 * LIMIT // 512 + 1, 0, False, False),
    (30_000, 64, 8500, 0, True, False), (9000, 64, 8500, 0, False, True), (30_000, 128, 8000, 7000, False, False), (9000, 1024, 2500, 0, False, False)])
def test_more_rows_than_the_batch_before_had(bags, dim, many, staging, inputs_ready, dirty):
    """Exactly as many missing rows as the index stream still fetches, one more, and far more, after batches of few."""
    class Uneven(TinyWorkload):
        def batch(self, t):
            ids, off = super().batch(t)
            fresh = many if t % 3 == 2 else 37
            ids = self.popular[ids % 50]
            # rows that no batch near this one has looked up, each once
            ids[:fresh] = self.rare[(np.arange(fresh) + t * many) % len(self.rare)]
            return ids, off

    w = Uneven(num_rows=60_000, dim=dim, cache_rows=many + 60, seed=bags + dim, multi_hot=False, bags=bags)
    by_rank = np.argsort(w.freq_rank)
    w.popular, w.rare = by_rank[:50], by_rank[many + 60:]
    run_parity_planned(w, 9, warm=True, dma_evict=True, staging_rows=staging, inputs_ready=inputs_ready, dirty_tracking=dirty)
