"""`-m gpu`: marks read chunk by chunk and counts added up over groups of tiles, against the oracle: tables that end at the edge of a
group of 16 tiles of 32768 ranks, popular rows among the highest ranks, none, a few and all of the marks read one and all."""
import pytest

from tests.parity import run_parity, run_parity_lookahead, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [524_288, 524_289, 1_048_577])
@pytest.mark.parametrize("dense", ["0", "4", "4096"])
@pytest.mark.parametrize("split_tiles", ["0", "1024"])
def test_mark_chunks(monkeypatch, rows, dense, split_tiles):
    monkeypatch.setenv("FC_MARK_DENSE", dense)
    monkeypatch.setenv("FC_PLAN_FOLD_TILES", split_tiles)
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=9000, seed=rows, multi_hot=False, bags=5000,
                     hot=[0, 255, 256, rows // 2, rows - 257, rows - 256, rows - 1], distinct_cap=4000)
    run_parity(w, 3, warm=False)
    run_parity_planned(w, 4, warm=True, dma_evict=True, inputs_ready=True)
    run_parity_lookahead(w, 4, warm=True)


@pytest.mark.parametrize("rows", [524_288, 524_289, 1_048_577])
@pytest.mark.parametrize("split_tiles", ["0", "1024"])
def test_bit_marks(monkeypatch, rows, split_tiles):
    """Where there is no room for a byte per row."""
    monkeypatch.setenv("FC_MARK_BYTES", "0")
    monkeypatch.setenv("FC_PLAN_FOLD_TILES", split_tiles)
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=9000, seed=rows + 1, multi_hot=False, bags=5000,
                     hot=[0, 31, 32, 255, rows // 2, rows - 257, rows - 1], distinct_cap=4000)
    run_parity(w, 3, warm=False)
    run_parity(w, 3, warm=True, dma_evict=True)
    run_parity_planned(w, 4, warm=True, dma_evict=True, inputs_ready=True)
    run_parity_lookahead(w, 4, warm=True)


@pytest.mark.parametrize("n", [(1 << 20) - 1, (1 << 20) + 1])
@pytest.mark.parametrize("dim", [4, 65])
def test_planned_batches_around_a_million_ids(n, dim):
    """Enqueued ahead of the decisions up to 2^20 ids and, where ids times columns stay below 2^26, beyond (65 columns: not beyond)."""
    w = TinyWorkload(num_rows=300_000, dim=dim, cache_rows=60_000, seed=n % 97 + dim, multi_hot=False, bags=n, distinct_cap=50_000)
    run_parity_planned(w, 3, warm=True, dma_evict=True, inputs_ready=True)
