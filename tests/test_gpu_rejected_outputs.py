"""A synchronous batch that holds an invalid query (a radius that is negative or not
a number, an infinite centre, an epoch that the index does not hold, a set that it
does not have) gives the error and leaves the caller's offsets and ids as they were,
at the sizes whose compaction is queued before the error is known and beyond; the
next valid batch in the same scratch is right."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_19891_amd import sfc, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 5000


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def outputs(m, cap):
    return dict(out_ids=torch.full((cap,), -7, dtype=torch.int32, device=DEV),
                out_offsets=torch.full((m + 1,), -7, dtype=torch.int64, device=DEV))


def rejected(call, m, cap):
    out = outputs(m, cap)
    with pytest.raises(sfc.SfcError) as err:
        call(out)
    assert err.value.status == sfc.SFC_ERR_INVALID
    assert (out["out_ids"] == -7).all() and (out["out_offsets"] == -7).all()


# 4097: the rows' scan in a launch of its own; 2^17 and one more: the last size queued
# as a whole, the first one whose rows are read first.
@pytest.mark.parametrize("m", [1, 300, 4097, 70_000, 1 << 17, (1 << 17) + 1])
@pytest.mark.parametrize("early_term", [False, True])
def test_outputs_stay(m, early_term):
    pts = workload.uniform_points(N, 71)
    q = workload.uniform_points(m, 72)
    d = np.full(m, workload.radius_for_count(4.0, N))
    want = oracle.query(oracle.build(pts, 0), q, d, 0, nthreads=8)
    idx = sfc.Index(dev(pts), sfc.MORTON, early_term=early_term)
    cap = len(want[1]) + 64
    for at in sorted({0, m // 2, m - 1}):
        for what in ("nan", "negative", "infinite"):
            bq, bd = q.copy(), d.copy()
            if what == "nan":
                bd[at] = np.nan
            elif what == "negative":
                bd[at] = -1.0
            else:
                bq[at, 1] = np.inf
            rejected(lambda out: idx.query(dev(bq), dev(bd), **out), m, cap)
    epochs = torch.zeros(m, dtype=torch.int32, device=DEV)
    epochs[m // 2] = 1
    rejected(lambda out: idx.query_epochs(dev(q), dev(d), epochs, **out), m, cap)
    off, ids = idx.query(dev(q), dev(d), **outputs(m, cap))
    assert torch.equal(off, dev(want[0].view(np.int64), torch.int64))
    assert torch.equal(ids, dev(want[1].view(np.int32), torch.int32))
    idx.close()


def test_outputs_stay_sets():
    pts, m = workload.uniform_points(N, 73), 500
    set_off = np.array([0, 1000, 1000, N], np.uint64)
    idx = sfc.Index(dev(pts), sfc.HILBERT, set_off=set_off)
    q, d = dev(workload.uniform_points(m, 74)), dev(np.full(m, 0.05))
    qset = torch.full((m,), 2, dtype=torch.int32, device=DEV)
    qset[m // 3] = 3
    rejected(lambda out: idx.query_sets(q, d, qset, **out), m, 64 * m)
    idx.close()
