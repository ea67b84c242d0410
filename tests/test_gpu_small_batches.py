"""`-m gpu`: batches that one workgroup indexes and sorts (up to 4096 ids, 2^20 rows, 2^16 slots), at the edges of its tiles
and of its range, against the oracle: every index decision and pooled row bit for bit."""
import pytest

from tests.parity import run_parity, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cache,bags", [
    (40, 40, 1), (40, 7, 6), (32768, 63, 63), (32769, 64, 64), (65536, 65, 65), (100_000, 1500, 1023), (100_001, 1025, 1024),
    (300_007, 15_001, 1025), (1_048_576, 65_536, 4095), (1_048_576, 65_537, 4096), (1_048_577, 5000, 4096), (262_145, 4500, 4097)])
@pytest.mark.parametrize("multi_hot,dma,warm", [(False, False, True), (False, True, False), (True, False, False), (True, True, True)])
def test_small_batches(rows, cache, bags, multi_hot, dma, warm):
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=cache, seed=rows + bags, multi_hot=multi_hot, bags=bags, max_bag=2,
                     hot=[1, 5, 17], distinct_cap=max(1, min(cache - 3, bags)))
    run_parity(w, 4, warm=warm, dma_evict=dma)
    if dma:
        run_parity_planned(w, 4, warm=warm, dma_evict=True, inputs_ready=multi_hot)


@pytest.mark.parametrize("cache,bags", [(1, 4097), (40, 10_239), (300, 10_240), (300, 10_241), (2, 6144), (3, 6145), (127, 8191), (128, 8193), (255, 4100), (256, 70_000), (511, 5000), (512, 2048 * 33 + 1)])
def test_sort_digit_widths(cache, bags):
    """Batches past the one-workgroup sort with digits of 1 to 9 bits and ragged last tiles, one and several supertiles."""
    w = TinyWorkload(num_rows=700, dim=4, cache_rows=cache, seed=cache, multi_hot=False, bags=bags, distinct_cap=cache)
    run_parity(w, 2, warm=True)
