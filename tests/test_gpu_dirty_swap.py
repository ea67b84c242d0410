"""`-m gpu`: FC_DIRTY_TRACK where rows change places in one kernel and clean victims are dropped by the slot assignment: phases of serving
and of training in turn, a flush between them or not, both transmitters (with FC_EVICT_DMA the kernel is used only while victims come out
clean and no block is on its way), batches that one workgroup indexes and larger ones, cold caches, more slot tiles than one."""
import pytest

from tests.parity import run_parity
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dma", [False, True])
@pytest.mark.parametrize("rows,cache,bags,dim", [(300, 37, 30, 3), (40_000, 1025, 1000, 20), (60_000, 5000, 9000, 6), (1_200_000, 1024, 700, 64), (90_000, 9000, 20_000, 4)])
@pytest.mark.parametrize("warm", [True, False])
@pytest.mark.parametrize("period,flush_at", [(1, ()), (3, ()), (4, (3, 7)), (100, ())])
def test_serving_and_training_in_turn(dma, rows, cache, bags, dim, warm, period, flush_at):
    w = TinyWorkload(num_rows=rows, dim=dim, cache_rows=cache, seed=rows + period, multi_hot=False, bags=bags, distinct_cap=max(1, cache * 2 // 3))
    run_parity(w, 10, warm=warm, dma_evict=dma, dirty_tracking=True, forward_only=lambda t: (t // period) % 2 == 0, flush_at=flush_at)
