"""`-m gpu`: sorts of up to 32 tiles of 2048 pairs, whose scatter kernel adds all tiles' counts up itself, and the first beyond, in the backward
pass that allocates nothing (which then needs scan kernels) and in the other: rows bit for bit the same, pooled rows those of the table."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [10_241, 12_288, 63_489, 65_536, 65_537])
@pytest.mark.parametrize("rows", [3, 500, 30_000, 400_000])
def test_one_supertile(n, rows):
    import torch
    from paper_2208_05321_amd import FreqCache
    dim = 8
    rng = np.random.default_rng([n, rows])
    ids = torch.from_numpy(np.minimum((rng.random(n) ** 2 * rows).astype(np.int64), rows - 1)).cuda()
    off = torch.arange(n + 1, device="cuda")
    grad = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    table = rng.standard_normal((rows, dim)).astype(np.float32)
    after = []
    for noalloc in (False, True):
        gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32), presort=not noalloc)
        gpu.host_weight()[:] = table
        gpu.warm()
        slots = gpu.prepare(ids, off)
        assert torch.equal(gpu.embedding_bag_fwd(slots, off).cpu(), torch.from_numpy(table)[ids.cpu()])
        (gpu.embedding_bag_bwd_sgd_noalloc if noalloc else gpu.embedding_bag_bwd_sgd)(slots, off, grad, 0.1)
        after.append(gpu.rows())
        gpu.check()
        gpu.close()
    assert np.array_equal(after[0], after[1])
    assert not np.array_equal(after[0], table)
