"""`-m gpu`: result arrays of freq_build where they start to travel in chunks (2,097,152 rows), around it and with ragged last
chunks, each output asked for or not, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2_097_151, 2_097_152, 2_097_153, 4_194_305, 6_000_001])
@pytest.mark.parametrize("with_counts", [True, False])
def test_results_in_chunks(rows, with_counts):
    import torch
    from paper_2208_05321_amd import FreqCounter
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    ids = (torch.rand(1_000_000, device="cuda", generator=g) ** 4 * rows).long().clamp_(max=rows - 1)
    f = FreqCounter(rows)
    f.add(ids)
    got = f.build(with_counts=with_counts)
    f.close()
    counts = np.bincount(ids.cpu().numpy(), minlength=rows)
    inv = np.argsort(-counts, kind="stable")
    rank = np.empty(rows, np.int64)
    rank[inv] = np.arange(rows)
    assert np.array_equal(got[0], rank) and np.array_equal(got[1], inv)
    if with_counts:
        assert np.array_equal(got[2], counts)
