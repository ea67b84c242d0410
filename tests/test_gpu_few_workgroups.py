"""`-m gpu`: batches that leave compute units idle: a lookup to a row-group in the forward pass (below 1024 workgroups of eight, checked on
either side), and in the backward pass runs that span many chunks of one workgroup, ending at, before and after the 64 chunks that a
mask holds, at its border and in the next workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(dim, ids, rows):
    import torch
    from oracle import Oracle
    from paper_2208_05321_amd import FreqCache
    n = len(ids)
    gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32))
    table = np.random.default_rng(7).standard_normal((rows, dim)).astype(np.float32)
    gpu.host_weight()[:] = table
    gpu.warm()
    orc = Oracle(np.arange(rows, dtype=np.int32), table.copy(), rows, warm=True)
    off = np.arange(n + 1, dtype=np.int64)
    ids_d, off_d = torch.from_numpy(ids).cuda(), torch.from_numpy(off).cuda()
    slots, so = gpu.prepare(ids_d, off_d), orc.prepare(ids, off)
    out = gpu.embedding_bag_fwd(slots, off_d)
    assert np.array_equal(out.cpu().numpy(), orc.embedding_bag_fwd(so, off))
    # gradients of small whole numbers and a rate of one: sums are exact in any order, so the rows agree bit for bit
    grad = np.random.default_rng(n).integers(-8, 9, (n, dim)).astype(np.float32)
    gpu.embedding_bag_bwd_sgd(slots, off_d, torch.from_numpy(grad).cuda(), 1.0)
    total = np.zeros((rows, dim))
    np.add.at(total, ids, grad)
    assert np.array_equal(gpu.rows(), table - total.astype(np.float32))
    gpu.check()
    gpu.close()
    orc.close()


@pytest.mark.parametrize("n", [1, 8183, 32_736, 32_737, 32_768, 32_769])
def test_forward_on_either_side_of_the_rule(n):
    _check(256, np.random.default_rng(n).integers(0, 700, n), 700)


@pytest.mark.parametrize("dim", [8, 9, 16, 64])
@pytest.mark.parametrize("head", [0, 3, 8])
@pytest.mark.parametrize("run", [5, 16, 64 * 8 - 8, 64 * 8 - 3, 64 * 8, 64 * 8 + 5, 128 * 8, 200 * 8 + 1, 511 * 8])
def test_runs_of_many_chunks(dim, head, run):
    """`head` lookups of other rows, the long run, and a tail: 512 chunks of 8 with 8 columns, one workgroup or several."""
    ids = np.concatenate([np.arange(head), np.full(run, 20), 21 + np.arange(max(0, 4096 - head - run)) // 3]).astype(np.int64)
    _check(dim, ids, 1500)


@pytest.mark.parametrize("dim,per_workgroup", [(256, 16), (50, 32), (16, 256)])
@pytest.mark.parametrize("over", [0, 1])
def test_bag_order_on_either_side_of_the_rule(dim, per_workgroup, over):
    """Serving without a sort: a bag to a row-group below 768 workgroups of four bags, four from there on."""
    import torch
    from paper_2208_05321_amd import FreqCache
    n, rows = 767 * per_workgroup + over, 900
    gpu = FreqCache(rows, dim, rows, np.arange(rows, dtype=np.int32), presort=False)
    table = np.random.default_rng(dim).standard_normal((rows, dim)).astype(np.float32)
    gpu.host_weight()[:] = table
    gpu.warm()
    ids = np.random.default_rng(n).integers(0, rows, n)
    off_d = torch.arange(n + 1, device="cuda")
    out = gpu.embedding_bag_fwd(gpu.prepare(torch.from_numpy(ids).cuda(), off_d), off_d)
    assert np.array_equal(out.cpu().numpy(), table[ids])
    gpu.check()
    gpu.close()
