"""`-m gpu`: the tables that a handle's first sort counts into are clear by then, also where nothing has been reserved and the sort runs
on a stream that nothing orders behind the null stream, where they are cleared.  (A race: handle after handle, each with its first
planned batch.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_first_planned_batches_of_many_handles():
    import torch
    from paper_2208_05321_amd import FreqCache
    n, rows, dim = 20_000, 60_000, 4
    off = torch.arange(n + 1, device="cuda")
    rng = np.random.default_rng(1)
    batches = [torch.from_numpy(rng.integers(0, 25_000, n)).cuda() for _ in range(2)]
    torch.cuda.synchronize()
    for k in range(20):
        gpu = FreqCache(rows, dim, 40_000, np.arange(rows, dtype=np.int32), dma_evict=True)
        gpu.host_weight()[:] = np.arange(rows, dtype=np.float32)[:, None]
        gpu.warm()
        gpu.prepare(batches[0], off)
        slots = gpu.plan_next(batches[1], off)
        gpu.advance()
        out = gpu.embedding_bag_fwd(slots, off)
        assert torch.equal(out, batches[1].float()[:, None].expand(-1, dim)), k
        gpu.check()
        gpu.close()
