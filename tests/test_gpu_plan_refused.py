"""`-m gpu`: cache_plan_next enqueues what depends on the decisions before it knows them; batches that are refused (each error)
or take another shape than the one before must leave the current batch, its sort and the cache as they were, raise no flag
of their own, and the next batch must come out right."""
import numpy as np
import pytest

from tests.parity import assert_close, compare_prepare
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bags,rows", [(300, 5000), (6000, 40_000), (9000, 1_200_000)])
@pytest.mark.parametrize("ready", [False, True])
def test_refused_plans_between_good_ones(bags, rows, ready, monkeypatch):
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache, FreqCacheError
    monkeypatch.setenv("FC_AHEAD_MISS_PCT", "100")
    cache_rows = bags + 100
    w = TinyWorkload(num_rows=rows, dim=8, cache_rows=cache_rows, seed=bags, multi_hot=False, bags=bags, distinct_cap=bags // 2)
    wm = TinyWorkload(num_rows=rows, dim=8, cache_rows=cache_rows, seed=bags, multi_hot=True, bags=bags // 3, max_bag=4, distinct_cap=bags // 2)
    dev = torch.device("cuda:0")
    gpu = FreqCache(rows, 8, cache_rows, w.freq_rank, dma_evict=True, inputs_ready=ready)
    host = gpu.host_weight()
    w.host_table(out=host)
    gpu.warm()
    orc = Oracle(w.freq_rank, host.copy(), cache_rows, warm=True)

    def up(*arrays):
        return [torch.from_numpy(a).to(dev) for a in arrays]

    def refused(kind):
        ids, off = w.batch(50)
        if kind == "BATCH_EXCEEDS_CACHE":
            ids = np.arange(cache_rows + 7, dtype=np.int64) % rows
            off = np.arange(len(ids) + 1, dtype=np.int64)
        elif kind == "ID_OUT_OF_RANGE":
            ids = ids.copy()
            ids[::7] = rows
            ids[3] = -1
        else:
            off = off.copy()
            off[2] = off[-1] + 5
        ids_d, off_d = up(ids, off)
        torch.cuda.synchronize()
        with pytest.raises(FreqCacheError) as e:
            gpu.plan_next(ids_d, off_d)
        assert e.value.name == kind

    shapes = [w, w, wm, w, wm, wm, w]
    data = []
    for t, x in enumerate(shapes):
        ids, off = x.batch(t)
        data.append((ids, off, x.grad(t, len(off) - 1), *up(ids, off, x.grad(t, len(off) - 1))))
    torch.cuda.synchronize()
    slots, so = gpu.prepare(data[0][3], data[0][4]), orc.prepare(data[0][0], data[0][1])
    for t in range(len(shapes)):
        ids, off, grad, ids_d, off_d, grad_d = data[t]
        out = gpu.embedding_bag_fwd(slots, off_d)
        for kind in ("BATCH_EXCEEDS_CACHE", "ID_OUT_OF_RANGE", "BAD_OFFSETS")[: 1 + t % 3]:
            refused(kind)                                    # between forward and backward: the sort must survive
        gpu.embedding_bag_bwd_sgd(slots, off_d, grad_d, 0.1)
        assert_close(out.cpu().numpy(), orc.embedding_bag_fwd(so, off), f"batch {t}: pooled")
        orc.embedding_bag_bwd_sgd(so, off, grad, 0.1)
        if t % 3 == 1:
            refused("ID_OUT_OF_RANGE")
        if t + 1 < len(shapes):
            so = orc.prepare(data[t + 1][0], data[t + 1][1])
            slots = gpu.plan_next(data[t + 1][3], data[t + 1][4])
            gpu.advance()
            compare_prepare(gpu, orc, slots.cpu().numpy(), so, t + 1)
    gpu.check()                                              # no flag was raised
    assert_close(gpu.rows(), orc.cache, "rows")
    gpu.flush()
    orc.flush()
    assert_close(host, orc.host, "host table")
    gpu.close()
    orc.close()


@pytest.mark.parametrize("bags,hot", [(300, 1), (300, 3), (9000, 1), (30_000, 1), (8000, 3)])
def test_a_refused_plan_leaves_the_callers_buffers_alone(bags, hot, monkeypatch):
    """The caller's stream is busy, so what was enqueued for the refused batch is still to run when the call has returned."""
    import torch
    from paper_2208_05321_amd import FreqCache, FreqCacheError
    monkeypatch.setenv("FC_AHEAD_MISS_PCT", "1000000")          # always ahead of the caller's stream
    n, rows = bags * hot, 8 * bags * hot
    cache_rows = n + 10
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, 4, cache_rows, np.arange(rows, dtype=np.int32), dma_evict=True, inputs_ready=True)
        gpu.host_weight()[:] = np.arange(rows, dtype=np.float32)[:, None]
        gpu.warm()
        gpu.reserve(rows, pipelined=True)
        off = torch.arange(bags + 1, device="cuda") * hot
        ids = [torch.arange(k * n, (k + 1) * n, device="cuda") for k in range(3)]
        much = torch.arange(cache_rows + hot, device="cuda")[: (cache_rows + hot) // hot * hot]
        far = ids[2].clone()
        far[5] = rows
        bad = off.clone()
        bad[3] = -1
        refusals = [(much, torch.arange(much.numel() // hot + 1, device="cuda") * hot, "BATCH_EXCEEDS_CACHE"),
                    (far, off, "ID_OUT_OF_RANGE"), (ids[2], bad, "BAD_OFFSETS")]
        torch.cuda.synchronize()
        gpu.prepare(ids[0], off)
        for t, (i, o, name) in enumerate(refusals):
            mine = torch.full((i.numel(),), 77, dtype=torch.int32, device="cuda")
            st.synchronize()
            torch.cuda._sleep(20_000_000)
            slots = gpu.plan_next(ids[(t + 1) % 3], off)
            gpu.advance()                                       # the next plan's sort comes behind the sleep
            with pytest.raises(FreqCacheError) as e:
                gpu.plan_next(i, o, out=mine)
            assert e.value.name == name
            torch.cuda.synchronize()
            assert bool((mine == 77).all())
            out = gpu.embedding_bag_fwd(slots, off)             # and the current batch is as it was
            want = ids[(t + 1) % 3].float().view(bags, hot)
            acc = torch.zeros(bags, device="cuda")
            for k in range(hot):
                acc = acc + want[:, k]
            assert torch.equal(out, acc[:, None].expand(-1, 4))
        gpu.check()
        gpu.close()
