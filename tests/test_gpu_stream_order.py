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
