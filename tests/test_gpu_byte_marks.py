"""`-m gpu`: byte marks against the oracle at the edges of a 32768-rank tile, and in turn on one handle, in every schedule, batches whose
marks are read one and all in different numbers of tiles (4 ranks per id, rounded up to tiles) and of the one-workgroup kind."""
import pytest

from tests.parity import run_parity, run_parity_lookahead, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


class Sizes(TinyWorkload):
    """Batch t has sizes[t % len] bags."""

    def __init__(self, sizes, **kw):
        super().__init__(bags=sizes[0], **kw)
        self.sizes = sizes

    def batch(self, t):
        self.bags = self.sizes[t % len(self.sizes)]
        return super().batch(t)


@pytest.mark.parametrize("rows", [32_767, 32_768, 32_769, 65_537, 1_048_576])
@pytest.mark.parametrize("multi_hot", [False, True])
def test_byte_marks(rows, multi_hot):
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=7000, seed=rows, multi_hot=multi_hot, bags=8300, max_bag=3, hot=[3, rows - 1],
                     distinct_cap=6500)
    run_parity(w, 3, warm=False)
    run_parity(w, 3, warm=True, dma_evict=True)


# 2, 1, 2, 2, 2, (one workgroup), 2, 2, 1, 2, 2, 3 tiles read one and all
SIZES = [12_000, 5000, 9375, 9374, 9376, 700, 12_000, 9000, 8192, 8193, 16_384, 16_385]


@pytest.mark.parametrize("rows", [300_000, 150_000])
def test_both_kinds_of_marks_in_turn(rows):
    w = Sizes(SIZES, num_rows=rows, dim=4, cache_rows=30_000, seed=7, multi_hot=False, distinct_cap=9000)
    run_parity(w, len(SIZES), warm=True)
    run_parity_planned(w, len(SIZES), warm=True, dma_evict=True, inputs_ready=True)
    run_parity_planned(w, len(SIZES), warm=False, dma_evict=False)
    for dma in (False, True):
        run_parity_lookahead(w, len(SIZES), warm=True, dma_evict=dma)
    tight = Sizes(SIZES, num_rows=rows, dim=4, cache_rows=13_000, seed=8, multi_hot=False, distinct_cap=9000)
    run_parity_lookahead(tight, len(SIZES), warm=True)                          # some look-aheads are refused


@pytest.mark.parametrize("fold", ["0", "1024"])
def test_dense_tiles_and_a_separate_plan(monkeypatch, fold):
    """A cold cache filled by a batch that misses half of every tile, then evictions of as many.  0: a tile to a workgroup of the
    emitting kernel (15,000 ranks of one tile in a list of 4096, round by round); 1024: eight workgroups to a tile."""
    monkeypatch.setenv("FC_PLAN_FOLD_TILES", fold)
    w = TinyWorkload(num_rows=70_000, dim=4, cache_rows=34_000, seed=9, multi_hot=False, bags=60_000, distinct_cap=33_000)
    run_parity(w, 4, warm=False)
    run_parity(w, 4, warm=True, dma_evict=True)
    tight = Sizes([60_000, 8500, 30_000], num_rows=70_000, dim=4, cache_rows=34_000, seed=10, multi_hot=False, distinct_cap=16_000)
    run_parity_lookahead(tight, 5, warm=False)
