"""`-m gpu`: what cache_plan_next makes the host wait for: its own planning kernels, and nothing that moves rows or trains."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

IDS, CACHE, DIM = 35_000, 40_000, 1024


def test_a_block_on_its_way_does_not_hold_up_the_next_plan(monkeypatch):
    """The controller of the early fetch reads the durations of finished block copies; asking about the one that the scatter
    threads are still waiting for makes the caller wait with them.  (On a handle that runs ahead of the caller's stream; one that
    does not may wait for a block, but only for an old one.)"""
    import torch
    from paper_2208_05321_amd import FreqCache
    monkeypatch.setenv("FC_AHEAD_MISS_PCT", "1000000")
    rows = 4 * IDS
    gpu = FreqCache(rows, DIM, CACHE, np.arange(rows, dtype=np.int32), dma_evict=True, inputs_ready=True)
    gpu.host_weight()[:] = 1.0
    gpu.warm()
    gpu.reserve(IDS, pipelined=True)
    off = torch.arange(IDS + 1, device="cuda")
    ids = [torch.arange(k * IDS, (k + 1) * IDS, device="cuda") for k in range(4)]       # every batch replaces most of the cache
    slots = [torch.empty(IDS, dtype=torch.int32, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    gpu.prepare(ids[0], off, out=slots[0])
    took = []
    for t in range(1, 13, 2):
        gpu.plan_next(ids[t % 4], off, out=slots[t & 1])
        gpu.advance()                                     # its evicted rows set out
        least = gpu.stats()["n_evict"] * DIM * 4 / 64e9   # seconds they need on the link
        time.sleep(0.0003)                                # the scatter threads wait for them by now
        a = time.perf_counter()
        gpu.plan_next(ids[(t + 1) % 4], off, out=slots[(t + 1) & 1])
        took.append((time.perf_counter() - a) / least)
        gpu.check()                                       # everything has arrived
    gpu.close()
    assert least > 1.8e-3
    assert min(took[2:]) < 0.4, took


@pytest.mark.parametrize("reserved", [True, False])
@pytest.mark.parametrize("n", [1000, 30_000])
def test_a_plan_after_a_plain_call_does_not_wait_for_the_current_batch(n, reserved):
    """Forward and backward of the current batch (a long kernel here) come after cache_prepare on the caller's stream; the planned
    batch's index work does not wait for them, on a handle that plans ahead or has announced it."""
    import torch
    from paper_2208_05321_amd import FreqCache
    rows = 8 * n
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        gpu = FreqCache(rows, 8, 2 * n, np.arange(rows, dtype=np.int32), dma_evict=True)
        gpu.host_weight()[:] = 1.0
        gpu.warm()
        off = torch.arange(n + 1, device="cuda")
        ids = [torch.arange(k * n, (k + 1) * n, device="cuda") for k in range(8)]
        slots = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        turns = range(1, 8, 2)
        if reserved:
            gpu.reserve(n, pipelined=True)
        else:                                             # what the first planned calls allocate is allocated
            for k in range(4):
                gpu.plan_next(ids[(2 * k + 5) % 8], off, out=slots[k & 1])
                gpu.advance()
            gpu.check()
        for t in turns:
            gpu.prepare(ids[t - 1], off, out=slots[0])
            torch.cuda._sleep(60_000_000)
            busy = torch.cuda.Event()
            busy.record(st)
            gpu.plan_next(ids[t], off, out=slots[1])
            assert not busy.query()
            gpu.advance()
            gpu.check()
        gpu.close()
