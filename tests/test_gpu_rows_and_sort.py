"""`-m gpu`: a batch of up to 10240 lookups is sorted by the first workgroup of the launch that brings its missing rows; both
transmitters, every vector width, one row to more than a round of the grid, at the ends of the sort's range and beside batches
without a missing row (whose sort goes alone)."""
import pytest

from tests.parity import run_parity
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


# 3 columns for accesses of one float: two orders of a sum differ by one rounding of its parts (2^-24 of 0.25 with these gradients and
# rate: 1.5e-8), which the row-wise limit of 1e-5 of the row's largest element plus 1e-9 covers unless all of a row lies below 1.4e-3.
# In rows of a single column a sum that cancels is such a row (seen: 4.6e-4 left, 1.5e-8 off), in wider ones all columns would have to.
@pytest.mark.parametrize("dim", [3, 6, 20, 516])
@pytest.mark.parametrize("rows,cache,bags,multi_hot", [(300, 2, 1, False), (40_000, 1100, 1024, False), (1_200_000, 4000, 4097, False),
                                                       (30_000, 8200, 10_240, False), (30_000, 9000, 4090, True), (5000, 5000, 700, False)])
@pytest.mark.parametrize("dma", [False, True])
def test_rows_and_sort(dim, rows, cache, bags, multi_hot, dma):
    w = TinyWorkload(num_rows=rows, dim=dim, cache_rows=cache, seed=dim + bags, multi_hot=multi_hot, bags=bags, distinct_cap=max(1, cache - 1))
    run_parity(w, 3, warm=True, dma_evict=dma, values_every=3)
