"""Which batches are searched in curve order, and their results: early termination
(a handle's first batch by a sample of its cells, the next ones by what the last one
had) and refined ranges through the learned index and the search tree (by the last
batch; the first through the tree from 2^20 queries on), among dense and nearly empty
batches in turn, recorded ones included; every result against the oracle.  Some
centres lie outside the domain, some radii are not valid."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_19891_amd import sfc, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N, M = (1 << 20) + 3, (1 << 17) + 1   # the least that is searched in curve order


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).to(DEV)


def ask(idx, q, d, want):
    """One batch, checked; whether its queries were put in order, and sampled."""
    sfc.profile_enable(True)
    try:
        sfc.profile_reset()
        off, ids = idx.query(q, d)
        ran = sfc.profile_read()
    finally:
        sfc.profile_enable(False)
    assert torch.equal(off, dev(want[0].view(np.int64), torch.int64))
    assert torch.equal(ids, dev(want[1].view(np.int32), torch.int32))
    return "query_order" in ran, "cells_sample" in ran


def batches(curve, m=M):
    """Points, and a dense and a nearly empty batch: (queries, radii, the oracle's)."""
    wl = workload.clustered_loguniform(n=N, m=m, curve=curve, seed=7, c_lo=60.0, c_hi=60.0)
    dense = wl.queries.copy()
    dense[::1000, 0] = -0.01
    dense[1::1000, 1] = 1.0
    empty = workload.uniform_points(m, 8)
    radii = np.full(m, workload.radius_for_count(1.0, N) / 16)
    built = oracle.build(wl.points, curve)
    return wl.points, [(q, d, oracle.query(built, q, d, curve, nthreads=8))
                       for q, d in ((dense, wl.delta), (empty, radii))]


@pytest.mark.parametrize("curve", [sfc.MORTON, sfc.HILBERT])
@pytest.mark.parametrize("refine", [False, True])
def test_early_termination(curve, refine):
    pts, (dense, empty) = batches(curve)
    dq, dd, dwant = dev(dense[0]), dev(dense[1]), dense[2]
    eq, ed, ewant = dev(empty[0]), dev(empty[1]), empty[2]
    for first in ("dense", "empty"):
        idx = sfc.Index(dev(pts), curve, refine=refine, early_term=True)
        # (the sampled order is queued and may do nothing on the device)
        if first == "dense":
            assert ask(idx, dq, dd, dwant) == (True, True)
        assert ask(idx, eq, ed, ewant) == (True, first == "empty")
        assert ask(idx, eq, ed, ewant) == (False, False)
        assert ask(idx, dq, dd, dwant) == (False, False)
        assert ask(idx, dq, dd, dwant) == (True, False)
        rows = idx.last_stats()["rows"]
        g = sfc.Graph.query(idx, dq, dd, max_rows=rows, ids_cap=len(dwant[1]))
        bad = dd.clone()
        bad[[0, M // 2, M - 1]] = float("nan")
        with pytest.raises(sfc.SfcError):
            idx.query(dq, bad)
        for _ in range(3):
            g.ids.fill_(-1)
            g.launch()
            off, ids = g.result()
            assert torch.equal(off, dev(dwant[0].view(np.int64), torch.int64))
            assert torch.equal(ids, dev(dwant[1].view(np.int32), torch.int32))
            idx.query(eq, ed)
        g.close()
        idx.close()
    # recorded before any batch: sampled at every replay
    idx = sfc.Index(dev(pts), curve, refine=refine, early_term=True)
    q, d = dq.clone(), dd.clone()
    g = sfc.Graph.query(idx, q, d, max_rows=rows, ids_cap=len(dwant[1]))
    for bq, bd, want in ((dq, dd, dwant), (eq, ed, ewant), (dq, dd, dwant)):
        q.copy_(bq)
        d.copy_(bd)
        g.launch()
        off, ids = g.result()
        assert torch.equal(off, dev(want[0].view(np.int64), torch.int64))
        assert torch.equal(ids[:len(want[1])], dev(want[1].view(np.int32), torch.int32))
    g.close()
    idx.close()


@pytest.mark.parametrize("search", [sfc.LEARNED, sfc.STREE])
@pytest.mark.parametrize("curve", [sfc.MORTON, sfc.HILBERT])
def test_refined(curve, search):
    pts, (dense, empty) = batches(curve)
    dq, dd, dwant = dev(dense[0]), dev(dense[1]), dense[2]
    eq, ed, ewant = dev(empty[0]), dev(empty[1]), empty[2]
    idx = sfc.Index(dev(pts), curve, search=search, refine=True)
    assert ask(idx, dq, dd, dwant) == (False, False)
    assert idx.last_stats()["candidates"] > 128 * M
    assert ask(idx, dq, dd, dwant) == (True, False)
    assert ask(idx, eq, ed, ewant) == (True, False)
    assert ask(idx, eq, ed, ewant) == (False, False)
    idx.close()
    idx = sfc.Index(dev(pts), curve, search=search, refine=False)
    for _ in range(2):
        assert ask(idx, dq, dd, dwant) == (False, False)
    idx.close()


def test_first_batch_through_the_tree():
    for m, ordered in (((1 << 20) - 1, False), (1 << 20, True)):
        pts, (_, empty) = batches(sfc.HILBERT, m)
        idx = sfc.Index(dev(pts), sfc.HILBERT, search=sfc.STREE, refine=True)
        q, d = dev(empty[0]), dev(empty[1])
        assert ask(idx, q, d, empty[2]) == (ordered, False)
        assert ask(idx, q, d, empty[2]) == (False, False)
        idx.close()
