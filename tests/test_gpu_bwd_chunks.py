"""`-m gpu`: the backward reduction where its cut changes: the last batch that fits one workgroup and the first that does not, the
last batch cut into chunks of 8 lookups and the first cut into chunks of 32 (for rows of every vector width, and for the widest, where
the limit is on the partial rows; rows of fewer than 8 columns are always cut into chunks of 32), a ragged last chunk, runs over many
chunks and workgroups, and bags of several lookups.

Bound, for every element: with u = 2^-24 a sum of K fp32 terms is off by at most (K - 1) u sum|g| in any order, the product with lr and
the subtraction add u each, so |row - (w - lr sum g)| <= (K + 2) u (|w| + lr sum|g|), up to a factor 1 + O(K u), taken as 1.01."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# dim -> lanes of a row: 1 -> 1, 8 -> 2, 7 -> 8, 16 -> 4, 9 -> 16, 50 and 128 -> 32, 63, 260 and 1024 -> 64
@pytest.mark.parametrize("dim,bags", [(1, 8191), (1, 8193), (16, 2048), (16, 2049), (50, 256), (50, 257), (128, 7), (128, 264), (1024, 128), (1024, 129),
                                      (260, 65536), (260, 65537), (1024, 32768), (1024, 32769),
                                      (7, 1024), (7, 1025), (8, 4096), (8, 4097), (9, 512), (9, 513), (63, 128), (63, 129), (9, 262_144), (9, 262_145), (63, 65_536), (63, 65_537)])
@pytest.mark.parametrize("hot", [0.0, 0.7])
def test_chunks(dim, bags, hot):
    import torch
    from paper_2208_05321_amd import FreqCache
    rows, lr = 700, np.float32(0.1)
    rng = np.random.default_rng([dim, bags, int(hot * 10)])
    gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32))
    w = rng.standard_normal((rows, dim), dtype=np.float32)
    gpu.host_weight()[:] = w
    gpu.warm()
    ids = rng.integers(0, rows, size=bags)
    ids = np.where(rng.random(bags) < hot, rng.integers(3, 5, size=bags), ids).astype(np.int64)
    grad = rng.standard_normal((bags, dim), dtype=np.float32)
    ids_d, off_d, grad_d = (torch.from_numpy(x).cuda() for x in (ids, np.arange(bags + 1, dtype=np.int64), grad))
    slots = gpu.prepare(ids_d, off_d)
    assert np.array_equal(slots.cpu().numpy(), ids)              # warm: slot s holds row s
    gpu.embedding_bag_bwd_sgd(slots, off_d, grad_d, float(lr))
    total, size = (torch.zeros(rows, dim, dtype=torch.float64, device="cuda") for _ in range(2))
    total.index_add_(0, ids_d, grad_d.double())
    size.index_add_(0, ids_d, grad_d.double().abs())
    want = w.astype(np.float64) - float(lr) * total.cpu().numpy()
    terms = np.bincount(ids, minlength=rows)[:, None]
    bound = 1.01 * (terms + 2) * 2.0 ** -24 * (np.abs(w) + float(lr) * size.cpu().numpy())
    got = gpu.rows()
    assert np.array_equal(got[terms[:, 0] == 0], w[terms[:, 0] == 0])
    assert (np.abs(got - want) <= bound).all()
    gpu.check()
    gpu.close()


@pytest.mark.parametrize("dim,n", [(9, 505), (9, 521), (16, 2041), (63, 4000), (128, 20_000)])
def test_chunks_of_bags(dim, n):
    """Fewer bags than lookups: a gradient row is read once per lookup of its bag."""
    import torch
    from paper_2208_05321_amd import FreqCache
    rows, lr = 300, np.float32(0.1)
    rng = np.random.default_rng([dim, n])
    gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32))
    w = rng.standard_normal((rows, dim), dtype=np.float32)
    gpu.host_weight()[:] = w
    gpu.warm()
    ids = np.where(rng.random(n) < 0.3, 7, rng.integers(0, rows, size=n)).astype(np.int64)
    off = np.concatenate([[0], np.sort(rng.integers(0, n + 1, size=n // 4)), [n]]).astype(np.int64)      # some bags are empty
    grad = rng.standard_normal((len(off) - 1, dim), dtype=np.float32)
    ids_d, off_d, grad_d = (torch.from_numpy(x).cuda() for x in (ids, off, grad))
    slots = gpu.prepare(ids_d, off_d)
    gpu.embedding_bag_bwd_sgd(slots, off_d, grad_d, float(lr))
    each = grad[np.repeat(np.arange(len(off) - 1), np.diff(off))].astype(np.float64)
    total, size = np.zeros((rows, dim)), np.zeros((rows, dim))
    np.add.at(total, ids, each)
    np.add.at(size, ids, np.abs(each))
    want = w.astype(np.float64) - float(lr) * total
    bound = 1.01 * (np.bincount(ids, minlength=rows)[:, None] + 2) * 2.0 ** -24 * (np.abs(w) + float(lr) * size)
    assert (np.abs(gpu.rows() - want) <= bound).all()
    gpu.check()
    gpu.close()
