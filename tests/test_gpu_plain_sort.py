"""`-m gpu`: a plain call's sort and its rows: beside each other on the default transmitter beyond 2^20 lookups, else one after the other."""
import numpy as np
import pytest

from tests.parity import run_parity
from tests.tiny_workload import TinyWorkload

pytestmark = pytest.mark.gpu

LIMIT = 1 << 20


@pytest.mark.parametrize("n,dma,beside", [(LIMIT, False, False), (LIMIT + 1, False, True), (LIMIT + 1, True, False)])
def test_what_runs_beside_the_rows(n, dma, beside, tmp_path, monkeypatch):
    import torch
    from paper_2208_05321_amd import FreqCache
    from tests.timeline_file import load_first_collection
    w = TinyWorkload(num_rows=400_000, dim=64, cache_rows=150_000, seed=n + dma, multi_hot=False, bags=n, distinct_cap=100_000)
    run_parity(w, 3, dma_evict=dma, values_every=0, fwd_exact_every=2)
    path = tmp_path / "timeline.txt"
    gpu = FreqCache(w.num_rows, w.dim, w.cache_rows, w.freq_rank, dma_evict=dma)
    gpu.host_weight()[:] = 1
    gpu.warm()
    dev = [tuple(torch.from_numpy(x).cuda() for x in w.batch(t)) for t in range(2)]
    gpu.prepare(*dev[0])
    gpu.check()
    monkeypatch.setenv("FC_TIMELINE", str(path))
    gpu.profile(True)
    gpu.prepare(*dev[1])
    gpu.check()
    gpu.profile_report()
    monkeypatch.delenv("FC_TIMELINE")
    gpu.profile(False)                                             # closes the file
    gpu.close()
    spans = load_first_collection(str(path))
    rows_in = max(b for a, b, name in spans if name == "miss_fill")
    sorting = min(a for a, b, name in spans if name == "sort_hist")
    assert (sorting < rows_in) == beside, spans
