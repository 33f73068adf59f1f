"""The rows that a batch is sized for before its count is known never fall as the
batch grows: a fresh handle's first batch of 20 rows a query is compacted once at
1024 queries and at the sizes past it, as long as its rows fit in those 2^16."""
import numpy as np
import pytest
import torch

from paper_2508_19891_amd import sfc, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,passes", [(1024, 1), (1025, 1), (2000, 1), (3276, 1), (3277, 2)])
def test_first_batch_compacted_once(m, passes):
    n = 20 * 64
    idx = sfc.Index(torch.as_tensor(workload.uniform_points(n, 81)).to(DEV), sfc.MORTON)
    q = torch.full((m, 2), 0.5, dtype=torch.float64, device=DEV)
    d = torch.full((m,), 2.0, dtype=torch.float64, device=DEV)
    ids = torch.empty(m * n, dtype=torch.int32, device=DEV)
    sfc.profile_enable(True)
    try:
        sfc.profile_reset()
        off, got = idx.query(q, d, out_ids=ids)
        launches = sfc.profile_read()
    finally:
        sfc.profile_enable(False)
    assert launches["compact_test"][0] == passes
    assert idx.last_stats()["rows"] == 20 * m
    assert np.array_equal(off.cpu().numpy(), np.arange(m + 1, dtype=np.int64) * n)
    assert (got.reshape(m, n) == got[:n]).all()
    idx.close()
