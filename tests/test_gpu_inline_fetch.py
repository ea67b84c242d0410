"""`-m gpu`: the fetch on the index stream, of rows whose lanes read 16, 8 and 4 bytes or are partly idle: against the oracle, and at a
rate over the link that does not depend on the form of the rows."""
import numpy as np
import pytest

from tests.parity import run_parity_planned
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 9, 33, 34, 65, 200, 257, 1023])
@pytest.mark.parametrize("bags,distinct", [(600, 300), (12_000, 1500)])
def test_forms_of_rows(dim, bags, distinct):
    w = TinyWorkload(num_rows=20 * distinct, dim=dim, cache_rows=distinct + 50, seed=bags + dim, multi_hot=False, bags=bags, distinct_cap=min(distinct, (3 << 19) // (4 * dim)))
    run_parity_planned(w, 4, warm=True, dma_evict=True)


def test_rate_of_odd_rows():
    import torch
    from paper_2208_05321_amd import FreqCache
    n, rows, cache, fresh = 40_000, 400_000, 50_000, 10_000
    us = {}
    for dim in (32, 33):
        gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32), dma_evict=True)
        gpu.host_weight()[:] = 1.0
        gpu.warm()
        off = torch.arange(n + 1, device="cuda")
        slots = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        for t in range(20):
            ids = torch.arange(n, device="cuda") % (cache - 2 * fresh)
            ids[:fresh] = cache + t * fresh + torch.arange(fresh, device="cuda")
            gpu.check()                                     # nothing else is on the link
            if t == 4:
                gpu.profile(True)
            gpu.plan_next(ids, off, out=slots[t & 1])
            gpu.check()
            assert gpu.stats()["n_miss"] == fresh
        rep = gpu.profile_report()["miss_fill"]
        us[dim] = rep["ms"] / rep["launches"] * 1e3
        gpu.close()
    assert us[33] < 1.5 * us[32], us
