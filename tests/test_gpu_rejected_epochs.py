"""Batches in which some queries ask for epochs that the index does not hold, among
valid ones: the error (or the flag of a queued batch), and then the right results of
valid batches in the same scratch, for every form of the search."""
import numpy as np
import pytest
import torch

from paper_2508_19891_amd import sfc, workload
from snapshots import Model

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
M = 3000


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def same(off, ids, want):
    total = len(want[1])
    assert torch.equal(off, dev(want[0].view(np.int64), torch.int64))
    assert torch.equal(ids[:total], dev(want[1].view(np.int32), torch.int32))


@pytest.mark.parametrize("search,early_term", [(sfc.BINARY, False), (sfc.BINARY, True),
                                               (sfc.STREE, False), (sfc.LEARNED, False)])
@pytest.mark.parametrize("refine", [False, True])
@pytest.mark.parametrize("curve", [sfc.MORTON, sfc.HILBERT])
def test_rejected_epochs(curve, refine, search, early_term):
    wl = workload.clustered_loguniform(n=20_000, m=M, curve=curve, seed=61)
    idx = sfc.Index(dev(wl.points), curve, search=search, refine=refine, early_term=early_term)
    idx.hold_epochs(True)
    model = Model(wl.points, hold=True)
    more = workload.uniform_points(4000, 62)
    for k in range(4):
        idx.insert(dev(more[1000 * k:1000 * (k + 1)]))
        model.insert(more[1000 * k:1000 * (k + 1)])
    idx.retire(2)
    model.retire(2)
    rng = np.random.default_rng(63)
    valid = rng.integers(2, model.epoch + 1, M)
    bad = valid.copy()
    for first, value in ((0, 1), (3, model.epoch + 1), (7, 0), (M - 1, -1)):
        bad[first::17] = value
    q, d = dev(wl.queries), dev(wl.delta)
    good_e, bad_e = dev(valid, torch.int32), dev(bad, torch.int32)
    want = model.reference(wl.queries, wl.delta, valid, curve)
    total = len(want[1])
    off = torch.empty(M + 1, dtype=torch.int64, device=DEV)
    ids = torch.empty(total, dtype=torch.int32, device=DEV)
    flags = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    max_rows = 64 * M
    stream = torch.cuda.Stream()
    scratch = torch.empty(idx.query_scratch_bytes(M, max_rows), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    for _ in range(2):
        with pytest.raises(sfc.SfcError):
            idx.query_epochs(q, d, bad_e)
        same(*idx.query_epochs(q, d, good_e), want)
        for e, flag in ((bad_e, 2), (good_e, 0)):
            idx.query_async(q, d, e, max_rows, off, ids, flags)
            torch.cuda.synchronize()
            assert int(flags[0]) == flag
        same(off, ids, want)
        for e, flag in ((bad_e, 2), (good_e, 0)):
            idx.query_async_on(stream, scratch, q, d, e, max_rows, off, ids, flags)
            torch.cuda.synchronize()
            assert int(flags[0]) == flag
        same(off, ids, want)
    idx.close()
