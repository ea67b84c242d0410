"""`-m gpu`: the bag that a sorted lookup is credited to, where a batch has as many lookups as bags without each bag holding its own:
at the edges of the one-workgroup sort's rounds and past it, sorted ahead of time and inside the backward call.

Bound as in test_gpu_bwd_chunks.py: (K + 2) u (|w| + lr sum|g|) for a row of K terms, u = 2^-24, times 1.01."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 64, 1025, 5120, 5121, 10_240, 10_241])
@pytest.mark.parametrize("shift", ["none", "first", "last"])         # which bag takes its neighbour's lookup
@pytest.mark.parametrize("noalloc", [False, True])
def test_bags_of_sorted_lookups(n, shift, noalloc):
    import torch
    from paper_2208_05321_amd import FreqCache
    rows, dim, lr = 500, 4, np.float32(0.1)
    rng = np.random.default_rng([n, len(shift)])
    w = rng.standard_normal((rows, dim), dtype=np.float32)
    gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32), presort=not noalloc)
    gpu.host_weight()[:] = w
    gpu.warm()
    ids = rng.integers(0, rows, size=n)
    off = np.arange(n + 1, dtype=np.int64)
    if shift == "first":
        off[1] = 2                       # bag 0: two lookups, bag 1: none
    elif shift == "last":
        off[n - 1] = n                   # the last bag: none
    grad = rng.standard_normal((n, dim), dtype=np.float32)
    ids_d, off_d, grad_d = (torch.from_numpy(x).cuda() for x in (ids, off, grad))
    slots = gpu.prepare(ids_d, off_d)
    (gpu.embedding_bag_bwd_sgd_noalloc if noalloc else gpu.embedding_bag_bwd_sgd)(slots, off_d, grad_d, float(lr))
    g = grad[np.repeat(np.arange(n), np.diff(off))].astype(np.float64)
    total, size = np.zeros((rows, dim)), np.zeros((rows, dim))
    np.add.at(total, ids, g)
    np.add.at(size, ids, np.abs(g))
    terms = np.bincount(ids, minlength=rows)[:, None]
    bound = 1.01 * (terms + 2) * 2.0 ** -24 * (np.abs(w) + float(lr) * size)
    assert (np.abs(gpu.rows() - (w.astype(np.float64) - float(lr) * total)) <= bound).all()
    gpu.check()
    gpu.close()
