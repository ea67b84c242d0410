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


@pytest.mark.parametrize("rows,cache,bags,dim", [(60_000, 900, 700, 32), (200_000, 15_000, 12_000, 16)])
def test_serving_after_training_with_the_block_transmitter(rows, cache, bags, dim):
    """Once the victims of earlier training have left and their blocks have arrived, rows change places in one kernel again: the first dirty victims
    after that are not gathered into a block."""
    import time

    import numpy as np
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache
    from tests.parity import assert_close
    fresh = bags // 2
    gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32), dma_evict=True, dirty_tracking=True)
    host = gpu.host_weight()
    host[:] = np.random.default_rng(1).standard_normal((rows, dim), dtype=np.float32)
    host_o = host.copy()
    gpu.warm()
    orc = Oracle(np.arange(rows, dtype=np.int32), host_o, cache, warm=True, dirty_tracking=True)
    off = np.arange(bags + 1, dtype=np.int64)
    off_d = torch.from_numpy(off).cuda()
    grad = np.ones((bags, dim), dtype=np.float32)
    grad_d = torch.from_numpy(grad).cuda()
    dirty = []
    for t in range(24):
        train = t < 6 or t == 20
        ids = np.arange(bags, dtype=np.int64) % (cache - 2 * fresh - 1)
        ids[:fresh] = cache + (t * fresh) % (rows - cache - fresh) + np.arange(fresh)
        if t == 20:
            time.sleep(0.1)                                        # the host threads are through with every block by now
        gpu.profile(t == 21)
        slots = gpu.prepare(torch.from_numpy(ids).cuda(), off_d)
        slots_o = orc.prepare(ids, off)
        assert np.array_equal(slots.cpu().numpy(), slots_o) and gpu.stats() == orc.stats(), t
        dirty.append(gpu.stats()["bytes_d2h"])
        if t == 21:
            rep = gpu.profile_report()
            gpu.profile(False)
        if train:
            gpu.embedding_bag_bwd_sgd(slots, off_d, grad_d, 0.5)
            orc.embedding_bag_bwd_sgd(slots_o, off, grad, 0.5)
    assert dirty[3] > 0 and dirty[20] == 0 and dirty[21] == fresh * dim * 4, dirty
    assert "miss_fill" in rep and "evict_gather" not in rep, rep
    assert_close(gpu.rows(), orc.cache, "cached rows")
    gpu.flush()
    orc.flush()
    assert_close(host, host_o, "host table")
    gpu.close()
    orc.close()


@pytest.mark.parametrize("dma", [False, True])
@pytest.mark.parametrize("rows,cache,bags,dim", [(40_000, 1025, 1000, 20), (90_000, 9000, 20_000, 4), (200_000, 9000, 12_000, 100)])
@pytest.mark.parametrize("free_running", [False, True])
def test_planned_and_plain_calls_in_turn(dma, rows, cache, bags, dim, free_running):
    """A dirty row that a plain call has stored in its place is fetched ahead of time by the planned batch that follows, and the other way round;
    phases of serving and of training, no flush between them."""
    import numpy as np
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache
    from tests.parity import STAT_FIELDS, assert_close
    w = TinyWorkload(num_rows=rows, dim=dim, cache_rows=cache, seed=rows + bags, multi_hot=False, bags=bags, distinct_cap=cache * 2 // 3)
    gpu = FreqCache(rows, dim, cache, w.freq_rank, dma_evict=dma, dirty_tracking=True)
    host = gpu.host_weight()
    w.host_table(out=host)
    host_o = host.copy()
    gpu.warm()
    orc = Oracle(w.freq_rank, host_o, cache, warm=True, dirty_tracking=True)
    data = [w.batch(t % 7) for t in range(28)]                     # batches come back: their rows have been evicted, some of them dirty, and return
    dev = [tuple(torch.from_numpy(x).cuda() for x in b) for b in data]
    rng = np.random.default_rng(5)
    planned = rng.random(28) < 0.5
    train = (np.arange(28) // 3) % 3 == 1
    later = []
    for t in range(28):
        ids, off = data[t]
        if planned[t]:
            slots = gpu.plan_next(*dev[t])
            gpu.advance()
        else:
            slots = gpu.prepare(*dev[t])
        slots_o = orc.prepare(ids, off)
        out = gpu.embedding_bag_fwd(slots, dev[t][1])
        later.append((t, slots, slots_o, out, orc.embedding_bag_fwd(slots_o, off)))
        if not free_running:
            assert {f: gpu.stats()[f] for f in STAT_FIELDS} == orc.stats(), t
        if train[t]:
            grad = w.grad(t, len(off) - 1)
            gpu.embedding_bag_bwd_sgd(slots, dev[t][1], torch.from_numpy(grad).cuda(), w.lr)
            orc.embedding_bag_bwd_sgd(slots_o, off, grad, w.lr)
    for t, slots, slots_o, out, out_o in later:
        assert np.array_equal(slots.cpu().numpy(), slots_o), t
        assert_close(out.cpu().numpy(), out_o, f"batch {t}: pooled output")
    assert_close(gpu.rows(), orc.cache, "cached rows")
    gpu.check()
    gpu.flush()
    orc.flush()
    assert_close(host, host_o, "host table")
    gpu.close()
    orc.close()
