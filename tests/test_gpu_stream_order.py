"""`-m gpu`: what a planned batch's index work has to wait for on the caller's stream when it runs ahead of it (FC_INPUTS_READY),
with the caller on a stream of his own and on the default one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def stream_of(kind):
    import torch
    return torch.cuda.Stream() if kind == "own" else torch.cuda.default_stream()


@pytest.mark.parametrize("kind", ["own", "default"])
@pytest.mark.parametrize("dma", [False, True])
def test_lists_outlive_the_row_movement_that_reads_them(kind, dma, monkeypatch):
    """Row movements of milliseconds (more rows than the block holds, so they all cross the link at cache_advance), plans of
    100 us: the lists that a movement reads are rewritten two plans later, the victims' ranks of a cache with blocks (which are
    kept per block, and no block is handed over here) by the very next one."""
    import torch
    from paper_2208_05321_amd import FreqCache
    monkeypatch.setenv("FC_AHEAD_MISS_PCT", "1000000")          # always ahead of the caller's stream
    n, rows, dim = 20_000, 80_000, 256
    st = stream_of(kind)
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, dim, n + 4000, np.arange(rows, dtype=np.int32), staging_rows=64, dma_evict=dma, inputs_ready=True)
        gpu.host_weight()[:] = np.arange(rows, dtype=np.float32)[:, None]
        gpu.warm()
        gpu.reserve(n, pipelined=True)
        off = torch.arange(n + 1, device="cuda")
        ids = [torch.arange(k * n, (k + 1) * n, device="cuda") for k in range(4)]
        slots = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        outs = [torch.empty(n, dim, device="cuda") for _ in range(9)]
        torch.cuda.synchronize()
        gpu.prepare(ids[0], off, out=slots[0])
        for t in range(9):
            gpu.embedding_bag_fwd(slots[t & 1], off, out=outs[t])
            gpu.plan_next(ids[(t + 1) % 4], off, out=slots[(t + 1) & 1])
            gpu.advance()
        gpu.check()
        gpu.flush()
        for t in range(9):
            assert torch.equal(outs[t], ids[t % 4].float()[:, None].expand(-1, dim)), f"batch {t}"
        assert np.array_equal(gpu.host_weight(), np.broadcast_to(np.arange(rows, dtype=np.float32)[:, None], (rows, dim)))
        gpu.close()


@pytest.mark.parametrize("planned", [False, True])
def test_rows_in_transit_when_a_batch_has_more_victims_than_a_block(planned):
    """Rows that left in a block and are missed by a batch whose victims are stored by kernel, through the blocks' memory."""
    import torch
    from paper_2208_05321_amd import FreqCache
    rows, dim, cache, S = 40_000, 8, 6000, 1000
    gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32), staging_rows=S, dma_evict=True)
    host = gpu.host_weight()
    host[:] = np.arange(rows, dtype=np.float32)[:, None]
    gpu.warm()

    def step(ranks):
        ids = torch.from_numpy(ranks).cuda()
        off = torch.arange(len(ranks) + 1, device="cuda")
        torch.cuda.synchronize()
        if planned:
            slots = gpu.plan_next(ids, off)
            gpu.advance()
        else:
            slots = gpu.prepare(ids, off)
        out = gpu.embedding_bag_fwd(slots, off).cpu().numpy()
        assert np.array_equal(out, np.broadcast_to(ranks.astype(np.float32)[:, None], out.shape))

    low = 5000                                              # ranks that stay throughout
    for first in range(4):                                  # every one of the four blocks in turn carries rows that come back
        for k in range(4 + first):
            new = np.arange(10_000 + 5000 * first + 700 * k, 10_000 + 5000 * first + 700 * (k + 1))
            step(np.concatenate([np.arange(low), new]))     # 700 rows in, 700 out in a block
        gone = np.arange(10_000 + 5000 * first, 10_000 + 5000 * first + 700 * (3 + first) - 1000)
        step(np.concatenate([np.arange(1500), gone, np.arange(30_000, 30_000 + 4200 - len(gone))]))
        step(np.arange(low))
    gpu.check()
    gpu.flush()
    assert np.array_equal(host, np.broadcast_to(np.arange(rows, dtype=np.float32)[:, None], host.shape))
    gpu.close()


@pytest.mark.parametrize("kind", ["own", "default"])
@pytest.mark.parametrize("dma", [False, True])
@pytest.mark.parametrize("bags", [5000, 100_000])
def test_plans_right_behind_refused_plain_calls(kind, dma, bags, monkeypatch):
    """A plain call that is refused returns while its last kernel still runs: it reads the bitmap and the counts."""
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache, FreqCacheError
    from tests.parity import compare_prepare
    from tests.tiny_workload import TinyWorkload
    monkeypatch.setenv("FC_AHEAD_MISS_PCT", "1000000")
    rows = 3_000_000
    w = TinyWorkload(num_rows=rows, dim=4, cache_rows=90_000, seed=bags, multi_hot=False, bags=bags, distinct_cap=80_000)
    st = stream_of(kind)
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, 4, w.cache_rows, w.freq_rank, dma_evict=dma, inputs_ready=True)
        host = gpu.host_weight()
        w.host_table(out=host)
        gpu.warm()
        gpu.reserve(200_000, pipelined=True)
        orc = Oracle(w.freq_rank, host.copy(), w.cache_rows, warm=True)
        good = [w.batch(t) for t in range(6)]
        on_gpu = [[torch.from_numpy(a).cuda() for a in b] for b in good]
        far = on_gpu[0][0].clone()
        far[7] = rows
        much = torch.arange(100_000, device="cuda") * 29
        much_off = torch.arange(100_001, device="cuda")
        torch.cuda.synchronize()
        for t in range(6):
            for ids, off, name in ((far, on_gpu[0][1], "ID_OUT_OF_RANGE"), (much, much_off, "BATCH_EXCEEDS_CACHE")):
                with pytest.raises(FreqCacheError) as e:
                    gpu.prepare(ids, off)
                assert e.value.name == name
                if name == ("ID_OUT_OF_RANGE" if t % 2 else "BATCH_EXCEEDS_CACHE"):
                    break
            slots = gpu.plan_next(*on_gpu[t])
            gpu.advance()
            compare_prepare(gpu, orc, slots.cpu().numpy(), orc.prepare(*good[t]), t)
        gpu.check()
        gpu.close()
        orc.close()
