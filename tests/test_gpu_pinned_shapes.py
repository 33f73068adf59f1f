"""A pinned launch shape does not send small batches back to reading their row count
in the middle: with pins for large and for small sizes, and after the autotuner, a
batch of 16 queries is still the same four launches (no scan of the rows by
itself), with the oracle's results."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_19891_amd import sfc, workload

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64).cuda()


def launches(idx, q, d, want):
    sfc.profile_reset()
    off, ids = idx.query(q, d)
    names = {k: v[0] for k, v in sfc.profile_read().items()}
    assert np.array_equal(off.cpu().numpy().view(np.uint64), want[0])
    assert np.array_equal(ids.cpu().numpy().view(np.uint32), want[1])
    return names


def test_small_batches_stay_unread():
    wl = workload.clustered_loguniform(n=50_000, m=16, curve=sfc.MORTON, seed=91)
    want = oracle.query(oracle.build(wl.points, sfc.MORTON), wl.queries, wl.delta, sfc.MORTON)
    q, d = dev(wl.queries), dev(wl.delta)
    idx = sfc.Index(dev(wl.points), sfc.MORTON)
    sfc.profile_enable(True)
    try:
        plain = launches(idx, q, d, want)
        assert "scan" not in plain
        for size in (1 << 25, 1 << 16, idx.last_stats()["rows"]):
            for shape in range(5):
                sfc.tune_pin(sfc.TUNE_TEST_SHAPE, size, shape)
                assert launches(idx, q, d, want) == plain
            sfc.tune_pin(sfc.TUNE_TEST_SHAPE, size, -1)
        sfc.autotune_query(idx, q, d)
        assert launches(idx, q, d, want) == plain
        fresh = sfc.Index(dev(wl.points), sfc.MORTON)
        assert launches(fresh, q, d, want) == plain
        fresh.close()
    finally:
        sfc.profile_enable(False)
        for size in (1 << 25, 1 << 16, idx.last_stats()["rows"]):
            sfc.tune_pin(sfc.TUNE_TEST_SHAPE, size, -1)
    idx.close()
