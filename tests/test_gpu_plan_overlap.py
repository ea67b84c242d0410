"""`-m gpu`: what of a planned batch runs beside what."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_rows_of_a_planned_batch_move_under_its_sort(tmp_path, monkeypatch):
    """Evicted rows are gathered as soon as the decisions are taken; a long sort (4 M lookups, few of them of missing rows) is still
    under way then."""
    import torch
    from paper_2208_05321_amd import FreqCache
    from tests.timeline_file import load_first_collection
    n, dim, rows, cache, popular, others = 1 << 22, 16, 200_000, 150_000, 80_000, 20_000
    path = tmp_path / "timeline.txt"
    monkeypatch.setenv("FC_TIMELINE", str(path))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32), dma_evict=True)
        gpu.host_weight()[:] = 1.0
        gpu.warm()
        gpu.reserve(n, pipelined=True)
        off = torch.arange(n + 1, device="cuda")
        k = torch.arange(n, device="cuda") % (popular + others)
        # the popular rows, and in turn either of two groups of rare ones, each of which takes the other's place
        ids = [torch.where(k < popular, k, k + rows - (1 + g) * others - popular) for g in range(2)]
        slots = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        gpu.prepare(ids[0], off, out=slots[0])
        steps = 4
        for t in range(1, 8):
            if t == 8 - steps:
                gpu.check()
                gpu.profile(True)
            gpu.plan_next(ids[t & 1], off, out=slots[t & 1])
            gpu.advance()
            gpu.check()                                   # everything has arrived before the next step
            stats = gpu.stats()
        gpu.profile_report()
        gpu.profile(False)
        monkeypatch.delenv("FC_TIMELINE")
        gpu.profile(False)                                # closes the file
        assert 0 < stats["n_evict"] * dim * 4 < 4 << 20, stats
        gpu.close()
    spans = load_first_collection(str(path))
    gathers = [a for a, b, name in spans if name == "evict_gather"]
    scatters = [b for a, b, name in spans if name == "sort_scatter"]
    assert len(gathers) == steps and len(scatters) % steps == 0 and scatters
    ends = scatters[len(scatters) // steps - 1::len(scatters) // steps]          # of each step's last pass
    # (behind the sort it can never be; a host that is held up may once be late with the gather)
    assert sum(a < b for a, b in zip(gathers, ends)) >= steps - 1, (gathers, ends)


@pytest.mark.parametrize("n", [10_000, 60_000])                   # sorted in the launch that fetches, and after it
def test_rows_leave_while_rows_arrive_after_a_batch_of_few(n, tmp_path, monkeypatch):
    """A batch with many missing rows after one with few: its victims are gathered while its rows are fetched, not behind them."""
    import torch
    from paper_2208_05321_amd import FreqCache
    dim, rows, cache, few, many, steps = 256, 700_000, 60_000, 100, n * 3 // 4, 4
    path = tmp_path / "timeline.txt"
    monkeypatch.setenv("FC_TIMELINE", str(path))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, dim, cache, np.arange(rows, dtype=np.int32), dma_evict=True)
        gpu.host_weight()[:] = 1.0
        gpu.warm()
        gpu.reserve(n, pipelined=True)
        off = torch.arange(n + 1, device="cuda")
        fresh = iter(range(cache, rows - many, many))
        slots = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        batches = []
        for t in range(2 * steps + 2):
            m = few if t % 2 == 0 else many
            ids = torch.arange(n, device="cuda") % (cache - many - 2 * few)
            ids[:m] = next(fresh) + torch.arange(m, device="cuda")
            batches.append(ids)
        gpu.prepare(batches[0], off, out=slots[0])
        for t in range(1, len(batches)):
            gpu.check()                                            # nothing is under way when the step begins
            gpu.profile(t >= 3 and t % 2 == 1)
            gpu.plan_next(batches[t], off, out=slots[t & 1])
            gpu.advance()
            assert gpu.stats()["n_miss"] == gpu.stats()["n_evict"] == (many if t % 2 else few)
        gpu.check()
        monkeypatch.delenv("FC_TIMELINE")
        gpu.profile(False)                                         # closes the file
        gpu.close()
    collections, cur = [], None
    for line in open(path):
        if line.startswith("#"):
            collections.append(cur := {"gather": [], "fill": []})
        elif line.startswith(("evict_gather", "miss_fill")):
            name, a, b = line.split()
            cur["gather" if name == "evict_gather" else "fill"].append((float(a), float(b)))
    done = [c for c in collections if c["gather"] and c["fill"]]
    assert len(done) >= steps - 1, collections
    # (a host that is held up may once be late with the gather)
    late = [c for c in done if c["gather"][0][0] > max(b for _, b in c["fill"])]
    assert len(late) <= 1, (late, done)
