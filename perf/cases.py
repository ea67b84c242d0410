"""Performance cases: what a training or serving program has the software cache do, call by call.

Every case goes through the public entry points (`FreqCache`, `FreqCounter`) on synthetic inputs made from a seed on
the GPU: `features` id columns concatenated into one table of `rows` rows, ids bounded-Zipf(`alpha`) per column, rows
ranked by popularity, a cache of `cache` rows, `samples` x `features` bags per batch.  The shapes are the ones that
workloads/gen.py defines (c1, c2, c2d32, c4, c5, avz), with fewer rows where the table would not fit pinned memory
three times over, plus small and odd ones.

One pass of a training case is one turn of the loop  fwd(t); bwd(t); prepare(t+1)  -- or, pipelined,
fwd(t); bwd(t); plan_next(t+1); advance()  -- started at bwd(t), so that it ends with the forward of batch t+1, whose
pooled rows carry the update that the pass has made.  `prepare` leaves batch 0 prepared and pooled.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2208_05321_amd import FreqCache, FreqCounter

LR = 0.01
RING = 4                 # batches of a state, taken in turn: a rare id of one batch has left the cache when it comes back
GRADS = 2                # upstream gradients of a state, taken in turn
PINNED_MOST = 8 << 30    # bytes of the host table


def _case(name, kind, rows, dim, features, samples, cache, alpha, bag=1, schedule="plain", transmitter="direct",
          inputs_ready=False, presort=True, dirty=False, noalloc=False, flush=False, chunks=1):
    c = dict(kind=kind, rows=rows, dim=dim, features=features, samples=samples, cache=cache, alpha=alpha, bag=bag,
             schedule=schedule, transmitter=transmitter, inputs_ready=inputs_ready, presort=presort, dirty=dirty,
             noalloc=noalloc, flush=flush, chunks=chunks)
    return {"name": name, **c} if name else c


def listed():
    piped = dict(schedule="pipelined", transmitter="dma", inputs_ready=True)
    return [
        # c1, the smallest configuration: a small model's or a unit-sized step, with the defaults of every option
        _case("train_c1", "train", 100_000, 16, 1, 1024, 1500, 1.1),
        # online inference: a request batch of 128 samples; no backward pass follows
        _case("serve_small", "serve", 1_000_000, 64, 26, 128, 15_000, 1.05, presort=False),
        # odd sizes throughout, the backward pass that allocates nothing, and a checkpoint (the table complete on the host)
        _case("train_odd_checkpoint", "train", 300_007, 50, 13, 777, 15_001, 1.05, presort=False, noalloc=True, flush=True),
        # an everyday click-model batch: 2048 samples, 64 columns
        _case("train_2k", "train", 4_000_000, 64, 26, 2048, 60_000, 1.05, **piped),
        # bulk scoring at c2's shape: victims are dropped, none is dirty
        _case("serve_c2", "serve", 10_000_000, 128, 26, 16_384, 150_000, 1.05, presort=False, dirty=True),
        # c2: the paper's dim and batch, 10M rows, 1.5% cache
        _case("train_c2", "train", 10_000_000, 128, 26, 16_384, 150_000, 1.05, **piped),
        # c2 as one of four ranks of a column split sees it
        _case("train_c2d32", "train", 10_000_000, 32, 26, 16_384, 150_000, 1.05, **piped),
        # avz, the paper's second dataset shape, plain schedule and default transmitter
        _case("train_avz_plain", "train", 9_445_823, 128, 13, 65_536, 141_687, 1.05),
        # c5: bags of about 20 lookups (multi-hot), wide rows
        _case("train_c5", "train", 8_000_000, 256, 8, 2048, 400_000, 1.05, bag=20, **piped),
        # c4's index work in full (100M rows, 1.5M slots, 1.7M ids), as one of eight ranks of a column split sees it
        _case("train_c4d16", "train", 100_000_000, 16, 26, 65_536, 1_500_000, 1.2, **piped),
        # c4's batch and row width: the largest
        _case("train_c4", "train", 16_000_000, 128, 26, 65_536, 240_000, 1.2, **piped),
        # the static module: ids of 8 batches counted, c2's rows ranked
        _case("static_c2", "static", 10_000_000, 0, 26, 16_384, 0, 1.05, chunks=8),
    ]


def draw(rng):
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("train", "train", "train", "train", "serve", "multi", "static"))
    features = rng.choice((1, 4, 8, 13, 26, rng.randint(2, 26)))
    if kind == "static":
        return _case(None, "static", logu(100_000, 20_000_000), 0, features, logu(256, 65_536), 0,
                     rng.choice((1.05, 1.1, 1.2)), chunks=rng.randint(1, 8))
    dim = rng.choice((16, 32, 64, 128, 128, 256, logu(8, 256)))
    bag = rng.randint(2, 30) if kind == "multi" else 1
    rows = min(logu(100_000, 60_000_000), PINNED_MOST // (4 * dim))
    samples = logu(64, 65_536)
    # no more lookups, and no more bytes of rows, than the largest listed case
    samples = max(1, min(samples, 1_700_000 // (features * bag), 200_000_000 // (features * bag * dim)))
    schedule = rng.choice(("plain", "pipelined"))
    transmitter = rng.choice(("direct", "dma")) if schedule == "plain" else "dma"
    c = _case(None, "serve" if kind == "serve" else "train", rows, dim, features, samples, 1, rng.choice((1.05, 1.1, 1.2)), bag=bag,
              schedule="plain" if kind == "serve" else schedule, transmitter=transmitter,
              inputs_ready=kind != "serve" and schedule == "pipelined", presort=kind != "serve",
              dirty=kind == "serve" and rng.random() < 0.5,
              noalloc=kind == "train" and schedule == "plain" and samples * features <= 200_000 and rng.random() < 0.3)
    if c["noalloc"]:
        c["presort"] = False
    # a batch has to fit the cache, with room for the spread of its distinct rows
    need = int(1.15 * _expected(c)[0]) + 256
    c["cache"] = min(rows, max(int(rows * rng.choice((0.005, 0.015, 0.05))), need))
    return c


# ---- distributions ---------------------------------------------------------------------------------------------------
def _cards(case):
    """Rows per id column: a geometric progression from 10 (one tiny column, a few huge ones) that sums to `rows`."""
    rows, f = case["rows"], case["features"]
    if f == 1:
        return np.array([rows], dtype=np.int64)
    lo, hi = 0.0, math.log(rows)
    for _ in range(60):
        mid = (lo + hi) / 2
        if 10 * np.exp(np.linspace(0, mid, f)).sum() < rows:
            lo = mid
        else:
            hi = mid
    c = np.maximum(1, np.floor(10 * np.exp(np.linspace(0, lo, f)))).astype(np.int64)
    c[-1] += rows - c.sum()
    return c


def _expected(case):
    """(distinct rows, missing rows) of a batch, expected; missing = distinct rows beyond the `cache` most popular."""
    s, e = case["samples"] * case["bag"], 1.0 - case["alpha"]
    ps, ns = [], []
    for k in _cards(case):
        edge = np.unique(np.floor(np.exp(np.linspace(0, math.log(k + 1.0), 400)))).astype(np.float64)
        a, b = edge[:-1], edge[1:]
        n = b - a
        ps.append((a ** e - b ** e) / (1.0 - (k + 1.0) ** e) / n)
        ns.append(n)
    p, n = np.concatenate(ps), np.concatenate(ns)
    seen = n * -np.expm1(s * np.log1p(-np.minimum(p, 1 - 1e-12)))
    o = np.argsort(-p)
    beyond = np.clip((np.cumsum(n[o]) - case["cache"]) / n[o], 0.0, 1.0)
    return float(seen.sum()), float((seen[o] * beyond).sum())


def _gen(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * seed + part)
    return g


def _bag_sizes(case, bags, g):
    """Poisson bag sizes in [1, 64], adjusted here and there by one so that every batch has bags x bag lookups."""
    size = torch.poisson(torch.full((bags,), float(case["bag"]), device="cuda"), generator=g).clamp_(1, 64).long()
    while True:
        d = bags * case["bag"] - int(size.sum())
        if d == 0:
            return size
        step = 1 if d > 0 else -1
        order = torch.randperm(bags, generator=g, device="cuda")
        order = order[(size[order] + step >= 1) & (size[order] + step <= 64)][:abs(d)]
        size[order] += step


def _ids(case, seed):
    """freq_rank int32[rows] and the ring's batches [(ids int64[n], offsets int64[bags + 1])], on the GPU."""
    g = _gen(seed, 1)
    cards = _cards(case)
    off = np.concatenate([[0], np.cumsum(cards)])
    e = 1.0 - case["alpha"]
    rows = case["rows"]
    perm = torch.empty(rows, dtype=torch.int64, device="cuda")         # popularity position (column by column) -> id
    score = torch.empty(rows, dtype=torch.float64, device="cuda")      # its probability, up to a factor
    for f, k in enumerate(cards):
        a, b = int(off[f]), int(off[f + 1])
        perm[a:b] = torch.randperm(int(k), generator=g, device="cuda") + a
        pos = torch.arange(1, int(k) + 1, dtype=torch.float64, device="cuda")
        score[a:b] = (pos + 0.5).pow_(-case["alpha"]) / (1.0 - (float(k) + 1.0) ** e)
    order = torch.argsort(score, descending=True)
    del score
    freq_rank = torch.empty(rows, dtype=torch.int32, device="cuda")
    freq_rank[perm[order]] = torch.arange(rows, dtype=torch.int32, device="cuda")
    del order
    fo = torch.from_numpy(off[:-1]).cuda()
    kk = torch.from_numpy(cards).cuda().double()
    bags = case["samples"] * case["features"]
    batches = []
    for _ in range(RING if case["kind"] != "static" else case["chunks"]):
        feat = torch.arange(bags, device="cuda") % case["features"]
        offsets = torch.arange(bags + 1, dtype=torch.int64, device="cuda")
        if case["bag"] > 1:
            size = _bag_sizes(case, bags, g)
            offsets[1:] = torch.cumsum(size, 0)
            feat = torch.repeat_interleave(feat, size)
        u = torch.rand(feat.numel(), dtype=torch.float64, device="cuda", generator=g)
        k1 = kk[feat]
        x = (((k1 + 1.0) ** e - 1.0) * u + 1.0) ** (1.0 / e)
        pos = torch.minimum(x.floor_().clamp_(min=1.0), k1).long() - 1
        batches.append((perm[fo[feat] + pos], offsets))
    return freq_rank, batches


def _table(case, seed):
    """The rank-ordered table's start values, fp32 [rows, dim], on the GPU."""
    return torch.rand(case["rows"], case["dim"], device="cuda", generator=_gen(seed, 2)).sub_(0.5).mul_(0.1)


def _grads(case, seed):
    bags, g = case["samples"] * case["features"], _gen(seed, 3)
    return [torch.randn(bags, case["dim"], device="cuda", generator=g) for _ in range(GRADS)]


# ---- the program -------------------------------------------------------------------------------------------------------
_stream = []


def _own_stream():
    """One stream for all work of this program, beside which the library's streams can run."""
    if not _stream:
        _stream.append(torch.cuda.Stream())
    return _stream[0]


def prepare(case, seed):
    freq_rank, batches = _ids(case, seed)
    if case["kind"] == "static":
        return {"case": case, "ids": [b[0] for b in batches], "stream": _own_stream()}
    host = torch.empty(case["rows"], case["dim"], dtype=torch.float32, pin_memory=True)
    host.copy_(_table(case, seed))
    torch.cuda.synchronize()
    st = _own_stream()
    cache = FreqCache(case["rows"], case["dim"], case["cache"], freq_rank.cpu().numpy(), host_weight=host, warm=True, stream=st,
                      staged=case["transmitter"] == "staged", dma_evict=case["transmitter"] == "dma", presort=case["presort"],
                      dirty_tracking=case["dirty"], inputs_ready=case["inputs_ready"])
    most = max(b[0].numel() for b in batches)
    bags = case["samples"] * case["features"]
    cache.reserve(most, pipelined=case["schedule"] == "pipelined")
    s = {"case": case, "cache": cache, "batches": batches, "t": 0, "host": host,
         "slots": [torch.empty(most, dtype=torch.int32, device="cuda") for _ in range(2)],
         "out": torch.empty(bags, case["dim"], dtype=torch.float32, device="cuda")}
    if case["kind"] == "train":
        s["grads"] = _grads(case, seed)
        torch.cuda.synchronize()
        ids, off = batches[0]
        slots = s["slots"][0][:ids.numel()]
        cache.prepare(ids, off, out=slots)
        cache.embedding_bag_fwd(slots, off, out=s["out"])
    torch.cuda.synchronize()
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "static":
        fc = FreqCounter(case["rows"], stream=state["stream"])
        for ids in state["ids"]:
            fc.add(ids)
        ranks = fc.build(with_counts=True)
        fc.close()
        return ranks
    cache, t = state["cache"], state["t"]
    state["t"] = t + 1
    if case["kind"] == "serve":
        ids, off = state["batches"][t % RING]
        slots = state["slots"][0][:ids.numel()]
        cache.prepare(ids, off, out=slots)
        return slots, cache.embedding_bag_fwd(slots, off, out=state["out"])
    ids, off = state["batches"][t % RING]
    slots = state["slots"][t & 1][:ids.numel()]
    backward = cache.embedding_bag_bwd_sgd_noalloc if case["noalloc"] else cache.embedding_bag_bwd_sgd
    backward(slots, off, state["grads"][t % GRADS], LR)
    ids, off = state["batches"][(t + 1) % RING]
    slots = state["slots"][(t + 1) & 1][:ids.numel()]
    if case["schedule"] == "pipelined":
        cache.plan_next(ids, off, out=slots)
        cache.advance()
    else:
        cache.prepare(ids, off, out=slots)
    pooled = cache.embedding_bag_fwd(slots, off, out=state["out"])
    if case["flush"]:
        cache.flush()
        return slots, pooled, state["host"]
    return slots, pooled


def work(case):
    ids = case["samples"] * case["features"] * case["bag"]
    if case["kind"] == "static":
        # the ids and the counters once; a sort's keys and values read and written once; three arrays to the host
        return {"bytes": 8.0 * ids * case["chunks"] + case["rows"] * (4.0 + 16.0 + 12.0), "flops": 0.0}
    bags, row = case["samples"] * case["features"], 4.0 * case["dim"]
    distinct, missing = _expected(case)
    # ids, ranks and slots; bag offsets; a distinct row read, a pooled row written; missing rows in, evicted rows out
    b = 16.0 * ids + 8.0 * bags + row * (distinct + bags) + 2 * row * missing
    f = float(case["dim"]) * ids
    if case["kind"] == "train":
        b += row * (bags + 2 * distinct)          # a gradient row read, a distinct row read and written
        f += case["dim"] * (ids + 2 * distinct)
    if case["flush"]:
        b += row * case["cache"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    # ranks, counts and one-hot rows that nothing has updated are copies; elsewhere fp32 sums, 0.9e-7 to 1.8e-7 off `exact`,
    # and another order of a popular row's gradients moves them by as much again
    if case["kind"] == "static" or (case["kind"] == "serve" and case["bag"] == 1):
        return "exact"
    return {"rel": 1e-6}


def exact(case, seed):
    if case["kind"] == "static":
        return None
    freq_rank, batches = _ids(case, seed)
    table = _table(case, seed)

    def ranks(b):
        return freq_rank[b[0]].long()

    def bag_of(b):
        n = b[0].numel()
        return torch.arange(n, device="cuda") if case["bag"] == 1 else torch.repeat_interleave(
            torch.arange(b[1].numel() - 1, device="cuda"), b[1][1:] - b[1][:-1])

    def pooled(b, rows_of):
        bags = b[1].numel() - 1
        if case["bag"] == 1:
            return rows_of(ranks(b))
        out = torch.zeros(bags, case["dim"], dtype=torch.float64, device="cuda")
        return out.index_add_(0, bag_of(b), rows_of(ranks(b)))

    if case["kind"] == "serve":
        return None, pooled(batches[0], lambda r: table[r].double())
    # the update of batch 0, kept for its distinct rows only, then batch 1's rows
    grad = _grads(case, seed)[0]
    uniq, inv = torch.unique(ranks(batches[0]), return_inverse=True)
    step = torch.zeros(uniq.numel(), case["dim"], dtype=torch.float64, device="cuda")
    step.index_add_(0, inv, grad.double()[bag_of(batches[0])])
    step *= float(np.float32(LR))
    place = torch.full((case["rows"],), -1, dtype=torch.int64, device="cuda")
    place[uniq] = torch.arange(uniq.numel(), device="cuda")

    def updated(r):
        at = place[r]
        hit = (at >= 0).unsqueeze(1)
        return table[r].double() - step[at.clamp(min=0)] * hit

    out = pooled(batches[1], updated)
    if not case["flush"]:
        return None, out
    table = table.double()
    table[uniq] -= step
    return None, out, table
