"""`-m gpu`: profiled items stand for one kind of work each, also for small batches, whose sort otherwise shares a launch with the rows and
whose evicted block is stored by its gather: the same items and launches as larger batches have, and the oracle's results."""
import numpy as np
import pytest

from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu

STEPS = 6


@pytest.mark.parametrize("bags", [700, 10_240])
@pytest.mark.parametrize("dma,planned", [(False, False), (True, False), (True, True)])
def test_items_of_small_batches(bags, dma, planned):
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache
    from tests.parity import assert_close
    w = TinyWorkload(num_rows=40_000, dim=20, cache_rows=700, seed=bags, multi_hot=False, bags=bags, distinct_cap=500)
    gpu = FreqCache(w.num_rows, w.dim, w.cache_rows, w.freq_rank, dma_evict=dma)
    host = gpu.host_weight()
    w.host_table(out=host)
    host_o = host.copy()
    gpu.warm()
    orc = Oracle(w.freq_rank, host_o, w.cache_rows, warm=True)
    for t in range(2 + STEPS):                                     # (the first planned batch goes by a guess)
        ids, off = w.batch(t)
        ids_d, off_d = torch.from_numpy(ids).cuda(), torch.from_numpy(off).cuda()
        gpu.check()
        if t == 2:
            gpu.profile(True)
        if planned:
            slots = gpu.plan_next(ids_d, off_d)
            gpu.advance()
        else:
            slots = gpu.prepare(ids_d, off_d)
        slots_o = orc.prepare(ids, off)
        assert np.array_equal(slots.cpu().numpy(), slots_o) and orc.stats()["n_evict"] > 0, t
        grad = w.grad(t, len(off) - 1)
        gpu.embedding_bag_bwd_sgd(slots, off_d, torch.from_numpy(grad).cuda(), w.lr)
        orc.embedding_bag_bwd_sgd(slots_o, off, grad, w.lr)
    gpu.check()
    rep = gpu.profile_report()
    gpu.profile(False)
    launches = {name: rep.get(name, {"launches": 0})["launches"] for name in ("miss_fill", "sort_scatter", "evict_gather", "d2h_block")}
    assert launches == {"miss_fill": STEPS, "sort_scatter": STEPS, "evict_gather": STEPS * dma, "d2h_block": STEPS * dma}, rep
    assert_close(gpu.rows(), orc.cache, "cached rows")
    gpu.flush()
    orc.flush()
    assert_close(host, host_o, "host table")
    gpu.close()
    orc.close()
