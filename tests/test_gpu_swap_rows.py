"""`-m gpu`: the default transmitter's row exchange (a slot's old row out, its new row in, in one kernel) where it can go wrong:
every vector width and rows wider than one pass of 64 lanes, a cold cache filling up (slots without an old row, then some with),
a cache thrashing in every batch, more rows than one round of the grid takes, and plain calls mixed with planned ones."""
import numpy as np
import pytest

from tests.parity import assert_close, compare_prepare, run_parity
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 2, 3, 20, 66, 128, 516])
@pytest.mark.parametrize("rows,cache,bags", [(200, 37, 30), (20_000, 6000, 4300)])
@pytest.mark.parametrize("warm", [True, False])
def test_swap_rows(dim, rows, cache, bags, warm):
    w = TinyWorkload(num_rows=rows, dim=dim, cache_rows=cache, seed=dim + rows, multi_hot=False, bags=bags, distinct_cap=cache - 5)
    run_parity(w, 4, warm=warm, flush_at=(1,), values_every=2)


def test_more_rows_than_one_round_of_the_grid():
    w = TinyWorkload(num_rows=90_000, dim=256, cache_rows=30_000, seed=3, multi_hot=False, bags=40_000, distinct_cap=29_000)
    run_parity(w, 3, warm=True, values_every=3)


@pytest.mark.parametrize("bags", [50, 5000])
def test_plain_and_planned_calls_in_turn(bags):
    """Events that a plain call leaves unrecorded are made good by the planned call that follows, in both orders."""
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache
    w = TinyWorkload(num_rows=9000, dim=32, cache_rows=3000, seed=bags, multi_hot=False, bags=bags, distinct_cap=2900)
    dev = torch.device("cuda:0")
    gpu = FreqCache(w.num_rows, w.dim, w.cache_rows, w.freq_rank)
    host = gpu.host_weight()
    w.host_table(out=host)
    gpu.warm()
    orc = Oracle(w.freq_rank, host.copy(), w.cache_rows, warm=True)
    data = []
    for t in range(12):
        ids, off = w.batch(t)
        data.append((ids, off, w.grad(t, bags), torch.from_numpy(ids).to(dev), torch.from_numpy(off).to(dev)))
    slots = gpu.prepare(data[0][3], data[0][4])
    so = orc.prepare(data[0][0], data[0][1])
    for t in range(11):
        ids, off, grad, ids_d, off_d = data[t]
        out = gpu.embedding_bag_fwd(slots, off_d)
        assert_close(out.cpu().numpy(), orc.embedding_bag_fwd(so, off), f"batch {t}")
        gpu.embedding_bag_bwd_sgd(slots, off_d, torch.from_numpy(grad).to(dev), w.lr)
        orc.embedding_bag_bwd_sgd(so, off, grad, w.lr)
        so = orc.prepare(data[t + 1][0], data[t + 1][1])
        if t % 4 in (1, 2):
            slots = gpu.plan_next(data[t + 1][3], data[t + 1][4])
            gpu.advance()
        else:
            slots = gpu.prepare(data[t + 1][3], data[t + 1][4])
        compare_prepare(gpu, orc, slots.cpu().numpy(), so, t + 1)
    gpu.check()
    gpu.flush()
    orc.flush()
    assert_close(host, orc.host, "host table")
    assert np.array_equal(gpu.state()[0], orc.slot_rank)
    gpu.close()
    orc.close()
