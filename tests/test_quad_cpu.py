"""A query's four search lanes as ordinary batches run them (query_quad.inc with
query_lane.h, learned.h, stree.h and curve.h) compiled as host C++ under the
address and undefined-behaviour sanitizers, on the CPU, four threads exchanging
words where the lanes do: the four places are written once each, whatever the box
and whether the query is rejected, and the places' index ranges, scanned with the
exact test, give the oracle's whole output id for id in curve order, for both
curves, the method's ranges and the refined cells, and every search."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from oracle import HILBERT, MORTON
from paper_2508_19891_amd import workload
from test_lane_cpu import learned_model, scan_slots

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_19891_amd", "csrc")
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if not os.path.isdir(ROCM_INCLUDE):
        pytest.skip("HIP headers not installed")
    exe = str(tmp_path_factory.mktemp("quad") / "quad_check")
    subprocess.check_call([
        "g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-pthread",
        "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-ffp-contract=off",
        "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE, "-I", CSRC,
        "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "cpu", "quad_check.cpp"),
        "-o", exe])
    return exe


def run(exe, tmp_path, keys, q, d, curve, refine, search=0, model=None, epochs=None, oldest=0,
        epoch=0):
    """(slots, rejected): every place's ranges, and per query whether it was rejected."""
    job, out = str(tmp_path / "job.bin"), str(tmp_path / "out.bin")
    n, m = len(keys), len(q)
    with open(job, "wb") as f:
        np.array([n, m, curve, int(refine), search, 32, 1, int(epochs is not None), oldest, epoch],
                 np.uint64).tofile(f)
        keys.astype(np.uint64).tofile(f)
        np.ascontiguousarray(q, np.float64).tofile(f)
        np.ascontiguousarray(d, np.float64).tofile(f)
        if epochs is not None:
            epochs.astype(np.uint32).tofile(f)
        if search == 1:
            xb, rt, lp, fk, pr, ps, dt = model
            for a in (xb, rt, lp, np.array([len(fk)], np.uint64), fk, pr, ps, dt):
                a.tofile(f)
    r = subprocess.run([exe, job, out], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    raw = np.fromfile(out, np.uint8)
    return (raw[:32 * 4 * m].view(np.uint64).reshape(m, 4, 4),
            raw[32 * 4 * m:].view(np.uint32).astype(bool))


def boxes(rng, pts, m):
    """Boxes of every level about cell corners, points and outside the square."""
    q = rng.random((m, 2))
    q[::4] = np.round(q[::4] * 8) / 8
    q[1::4] = pts[rng.integers(0, len(pts), len(q[1::4]))]
    d = 2.0 ** rng.uniform(-34, 1, m)
    d[::3] = 2.0 ** rng.uniform(-6, 0.5, len(d[::3]))
    edge = [[-0.5, 0.5], [0.5, 0.5], [1.5, 1.5], [1.0 - 2.0 ** -53, 1.0 - 2.0 ** -53], [0.0, 0.0],
            [0.25, 0.75], [1.0, 1.0], [5.0, 5.0]]
    q[:8] = edge
    d[:8] = [0.6, 2.0, 0.01, 1e-12, 0.0, 1e-300, 2.0 ** -32, 0.1]
    return q, d


@pytest.mark.parametrize("search", [0, 1, 2])
@pytest.mark.parametrize("refine", [False, True])
@pytest.mark.parametrize("curve", [MORTON, HILBERT])
def test_quad_matches_oracle(harness, tmp_path, curve, refine, search):
    rng = np.random.default_rng(100 * curve + 10 * refine + search)
    wl = workload.clustered_loguniform(n=20_000, m=1200, curve=curve, seed=21)
    q, d = boxes(rng, wl.points, 1200)
    q, d = np.concatenate([q, wl.queries]), np.concatenate([d, wl.delta])
    index = oracle.build(wl.points, curve)
    model = learned_model(index[0], rng) if search == 1 else None
    slots, rejected = run(harness, tmp_path, index[0], q, d, curve, refine, search, model)
    assert not rejected.any()
    got, want = scan_slots(index, q, d, slots, refine), oracle.query(index, q, d, curve, nthreads=4)
    assert np.array_equal(got[0], want[0])
    assert np.array_equal(got[1], want[1])


@pytest.mark.parametrize("refine", [False, True])
@pytest.mark.parametrize("curve", [MORTON, HILBERT])
def test_rejected_queries(harness, tmp_path, curve, refine):
    """Epochs outside the queryable ones, radii and centres that are not finite
    numbers (or negative) among valid queries: all four lanes reject, and leave four
    empty places; the others' are the oracle's."""
    rng = np.random.default_rng(40 + 2 * curve + refine)
    pts = rng.random((5000, 2))
    m = 1000
    q, d = boxes(rng, pts, m)
    epochs = rng.integers(3, 8, m)
    bad = np.zeros(m, bool)
    for first, value in ((10, 2), (11, 8), (12, 0), (13, 0xFFFFFFFF)):
        epochs[first::20] = value
        bad[first::20] = True
    d[14::20], d[15::20], q[16::20, 0], q[17::20, 1] = np.nan, -1.0, np.inf, np.nan
    for first in (14, 15, 16, 17):
        bad[first::20] = True
    index = oracle.build(pts, curve)
    slots, rejected = run(harness, tmp_path, index[0], q, d, curve, refine, epochs=epochs,
                          oldest=3, epoch=7)
    assert np.array_equal(rejected, bad)
    assert (slots[bad] == 0).all()
    ok = ~bad
    got = scan_slots(index, q[ok], d[ok], slots[ok], refine)
    want = oracle.query(index, q[ok], d[ok], curve, nthreads=4)
    assert np.array_equal(got[0], want[0])
    assert np.array_equal(got[1], want[1])
