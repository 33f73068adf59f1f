"""Construction of up to 2^16 points (one sorted run per workgroup, then every
element's rank in the others) gives the oracle's arrays: sizes about the rows of
a workgroup, the runs and the limit; spread, clustered and equal points; a
recorded construction; insertions."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_19891_amd import sfc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64).to(DEV)


def points(kind, n, dim, rng):
    if kind == "spread":
        return rng.random((n, dim))
    if kind == "edges":   # the first and the last cell, many times
        return np.where(rng.random((n, dim)) < 0.5, 0.0, 1.0 - 2.0 ** -53)
    p = 0.3 + 2.0 ** -18 * rng.random((n, dim))   # few top bits vary, long runs of equal ones
    p[::3] = p[0]
    return p


def arrays(idx):
    keys, ids, _ = idx.sorted_arrays()
    return keys.cpu().numpy().view(np.uint64), ids.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("kind", ["spread", "edges", "tight"])
@pytest.mark.parametrize("n", [1, 511, 513, 1024, 1025, 2049, 16384, 16385, 20_003, 65535, 65536,
                               65537])
def test_small_construction(n, kind):
    for curve in (sfc.MORTON, sfc.HILBERT, sfc.MORTON3):
        dim = 3 if curve == sfc.MORTON3 else 2
        pts = points(kind, n, dim, np.random.default_rng(n))
        built = oracle.build3(pts) if dim == 3 else oracle.build(pts, curve)
        idx = sfc.Index(dev(pts), curve)
        for _ in range(2):
            keys, ids = arrays(idx)
            assert np.array_equal(keys, built[0]) and np.array_equal(ids, built[1])
            g = sfc.Graph.build(idx, dev(pts))   # then once more, recorded
            g.launch()
            g.wait()
            g.close()
        idx.close()


@pytest.mark.parametrize("k", [1, 1023, 1025, 30_000, 65536, 65537])
def test_small_insertions(k):
    rng = np.random.default_rng(k)
    for curve in (sfc.MORTON, sfc.HILBERT):
        base = rng.random((5000, 2))
        new = rng.random((k, 2))
        new[::7] = base[rng.integers(0, 5000, len(new[::7]))]   # equal keys, new ids after old
        idx = sfc.Index(dev(base), curve)
        idx.insert(dev(new))
        keys, ids = arrays(idx)
        want = oracle.build(np.concatenate([base, new]), curve)
        assert np.array_equal(keys, want[0]) and np.array_equal(ids, want[1])
        bad = new.copy()
        bad[k // 2, 0] = 1.0
        with pytest.raises(sfc.DomainError):
            idx.insert(dev(bad))
        assert np.array_equal(arrays(idx)[0], want[0])
        idx.close()
