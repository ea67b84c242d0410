"""`-m gpu`: the general index kernels on the batches that one workgroup takes by default: random mixes of all calls, and caches
that thrash (rows that leave with one batch and are missed by the next, in transit or not), where their decisions go wrong first."""
import pytest

from tests import test_gpu_sequences
from tests.parity import run_parity, run_parity_lookahead, run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["0", "1024"], autouse=True)
def general_kernels(request, monkeypatch):
    monkeypatch.setenv("FC_SMALL_INDEX", "0")
    monkeypatch.setenv("FC_PLAN_FOLD_TILES", request.param)


@pytest.mark.parametrize("seed,dma,dirty,staging_rows", [(0, True, False, 0), (1, False, False, 0), (2, True, True, 0), (3, False, True, 0),
                                                         (4, True, False, 40), (5, True, True, 40), (6, True, False, 0), (7, True, True, 0)])
def test_random_call_sequences(seed, dma, dirty, staging_rows):
    test_gpu_sequences.test_random_call_sequences(seed, dma, dirty, staging_rows)


@pytest.mark.parametrize("rows", [900, 9000])
@pytest.mark.parametrize("dma", [True, False])
@pytest.mark.parametrize("free", [True, False])
def test_thrashing(rows, dma, free):
    w = TinyWorkload(num_rows=rows, dim=64, cache_rows=48, seed=21, multi_hot=True, bags=24, max_bag=3, distinct_cap=40)
    for ready in (False, True):
        run_parity_planned(w, 40, warm=True, dma_evict=dma, free_running=free, inputs_ready=ready)
        run_parity_planned(w, 24, warm=False, dma_evict=dma, free_running=free, inputs_ready=ready, staging_rows=16)
    run_parity_planned(w, 24, warm=True, dma_evict=dma, free_running=free, inputs_ready=True, miss_dma=True)
    run_parity(w, 12, warm=True, dma_evict=dma)
    run_parity_lookahead(w, 12, warm=True, dma_evict=dma)
