"""`-m gpu`: the largest batches that one workgroup indexes at the largest bitmap and slot count, and the first that no longer fit its LDS
(2 bytes an id beside 144 KB of bitmap and counts and 8 KB of slot masks), against the oracle, with batches that miss every row."""
import pytest

from tests.parity import run_parity, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cache,bags", [(65_536, 3584), (65_536, 3585), (8192, 4096), (4096, 4096), (4097, 1)])
@pytest.mark.parametrize("dma", [False, True])
def test_small_limits(cache, bags, dma):
    w = TinyWorkload(num_rows=1_048_576, dim=4, cache_rows=cache, seed=cache + bags, multi_hot=False, bags=bags, distinct_cap=bags)
    run_parity(w, 4, warm=False, dma_evict=dma)
    if dma:
        run_parity_planned(w, 5, warm=True, dma_evict=True, inputs_ready=True)
