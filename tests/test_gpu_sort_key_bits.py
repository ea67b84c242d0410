"""`-m gpu`: the one-workgroup sort holds key and lookup number in 32 bits: caches whose slots take the most bits that a batch's size leaves, and
one more (the general sort)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cache", [(1, (1 << 22) - 1), (1024, (1 << 22) - 1), (1024, 1 << 22), (1025, (1 << 21) - 1), (1025, 1 << 21), (4096, (1 << 20) - 1), (4097, 1 << 20),
                                     (10_240, (1 << 18) - 1), (10_240, 1 << 18)])
@pytest.mark.parametrize("hot", [0.0, 0.8])
def test_widest_keys(n, cache, hot):
    import torch
    from paper_2208_05321_amd import FreqCache
    dim, rows = 4, cache + 10
    rng = np.random.default_rng([n, cache])
    ids = np.where(rng.random(n) < hot, cache - 1 - rng.integers(0, 3, n), rng.integers(0, cache, n)).astype(np.int64)
    ids[-1] = cache - 1                                    # the largest slot
    gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32))
    gpu.host_weight()[:] = np.arange(rows, dtype=np.float32)[:, None] % 4096
    gpu.warm()
    off = torch.arange(n + 1, device="cuda")
    slots = gpu.prepare(torch.from_numpy(ids).cuda(), off)
    assert np.array_equal(slots.cpu().numpy(), ids)        # warm: slot s holds row s
    out = gpu.embedding_bag_fwd(slots, off)
    assert np.array_equal(out.cpu().numpy()[:, 0], ids % 4096)
    # whole gradients and a rate of one: the sums are exact in any order
    grad = rng.integers(-8, 9, (n, dim)).astype(np.float32)
    gpu.embedding_bag_bwd_sgd(slots, off, torch.from_numpy(grad).cuda(), 1.0)
    want = np.repeat((np.arange(cache) % 4096).astype(np.float64)[:, None], dim, 1)
    np.subtract.at(want, ids, grad)
    assert np.array_equal(gpu.rows(), want)
    gpu.check()
    gpu.close()
