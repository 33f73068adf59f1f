"""The chunked sort without point sets at more than 2^16 points, where builds take it
(smaller ones sort in two launches): last chunks on both sides of the stride (2048)
and of the capacity (4096), runs of equal top 32 bits up to the length that always
fits and beyond it, the fallback, and recorded builds with the fallback on the
device; every build also shows the kernels of the sort that it is meant to test."""
import numpy as np
import pytest
import torch

import oracle
from oracle import HILBERT, MORTON
from paper_2508_19891_amd import sfc
from test_gpu_sort_paths import M3, cell_run, dev, expected

pytestmark = pytest.mark.gpu
SMALL = 1 << 16   # builds of up to this many points sort in two launches


def check(pts, curve, fallback):
    sfc.profile_enable(True)
    try:
        sfc.profile_reset()
        idx = sfc.Index(dev(pts), curve=curve)
        ran = sfc.profile_read()
    finally:
        sfc.profile_enable(False)
    fell = sfc.debug_sort_path(-1)
    small = len(pts) <= SMALL
    assert ("small_runs" in ran) == small and ("chunk_sort" in ran) == (not small)
    # the passes over the top 32 bits, and the plain sort's eight behind them
    assert small or ran["scatter_pass"][0] == (12 if fell else 4)
    cells = idx.cells().cpu().numpy().view(np.uint64)
    keys, ids, _ = idx.sorted_arrays()
    k, i, c = expected(pts, curve)
    assert np.array_equal(keys.cpu().numpy().view(np.uint64), k)
    assert np.array_equal(ids.cpu().numpy().view(np.uint32), i)
    assert np.array_equal(cells, c)
    assert fallback is None or fell == fallback
    idx.close()


@pytest.mark.parametrize("curve", [MORTON, HILBERT, M3])
@pytest.mark.parametrize("n", [SMALL - 1, SMALL, SMALL + 1, SMALL + 2047, SMALL + 2048,
                               SMALL + 2049, SMALL + 4095, SMALL + 4096, SMALL + 4097,
                               SMALL + 12289])
def test_sizes(curve, n):
    rng = np.random.default_rng(n * 3 + curve)
    check(rng.random((n, 3 if curve == M3 else 2)), curve, 0)


@pytest.mark.parametrize("curve", [MORTON, HILBERT, M3])
@pytest.mark.parametrize("run", [1, 64, 65, 700, 2048])
def test_runs_that_always_fit(curve, run):
    """12 runs of equal top bits anywhere relative to the stride."""
    rng = np.random.default_rng(run + 17 * curve)
    dim = 3 if curve == M3 else 2
    pts = np.concatenate([rng.random((SMALL, dim))] + [cell_run(rng, run, dim) for _ in range(12)])
    check(pts[rng.permutation(len(pts))], curve, 0)


@pytest.mark.parametrize("curve", [MORTON, HILBERT, M3])
@pytest.mark.parametrize("runs,fallback", [((2100, 3000, 3500, 4000, 4096, 2600), None),
                                           ((4097,), 1), ((9000,), 1)])
def test_long_runs(curve, runs, fallback):
    """Runs past the stride fit or not by where the chunks start; past the capacity
    (equal keys too) they fall back."""
    rng = np.random.default_rng(99 + curve + len(runs))
    dim = 3 if curve == M3 else 2
    pts = np.concatenate([rng.random((70_000, dim))] + [cell_run(rng, s, dim) for s in runs] +
                         ([np.tile(rng.random((1, dim)), (5000, 1))] if runs == (9000,) else []))
    check(pts[rng.permutation(len(pts))], curve, fallback)


@pytest.mark.parametrize("curve", [MORTON, HILBERT, M3])
def test_recorded_build_falls_back_on_the_device(curve):
    """Replays on points that fit the chunks and on points that do not."""
    rng = np.random.default_rng(51 + curve)
    dim = 3 if curve == M3 else 2
    fit = rng.random((SMALL + 4321, dim))
    long_run = fit.copy()
    long_run[:9000] = cell_run(rng, 9000, dim)
    pts = dev(fit)
    idx = sfc.Index(pts, curve)
    gb = sfc.Graph.build(idx, pts)
    for rep, data in enumerate((long_run, fit, long_run, fit)):
        pts.copy_(dev(data))
        gb.launch()
        gb.wait()
        keys, ids, xy = idx.sorted_arrays()
        k, i, x = oracle.build3(data) if curve == M3 else oracle.build(data, curve)
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), k), rep
        assert np.array_equal(ids.cpu().numpy().view(np.uint32), i), rep
        assert np.array_equal(xy.cpu().numpy(), x), rep
    gb.close()
    idx.close()
