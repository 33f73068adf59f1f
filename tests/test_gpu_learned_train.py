"""The router's training step on the matrix cores: gradients at batch sizes on
and around its 16-sample tiles against FP64, and training itself against
the plain binary32 loop."""
import numpy as np
import pytest
import torch

import oracle
from oracle import learned as ref
from paper_2508_19891_amd import sfc, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cnt", [1, 2, 15, 16, 17, 63, 64, 65, 112, 113, 127, 128])
def test_gradient_at_tile_edges(cnt):
    rng = np.random.default_rng(cnt)
    p = ref.quantile_init(np.sort(rng.random(4096)))
    p = (p + 0.05 * rng.standard_normal(p.size)).astype(np.float32)
    x = (rng.integers(0, 1 << 24, cnt) / 2.0 ** 24).astype(np.float32)
    t = rng.random(cnt).astype(np.float32)
    g, loss = sfc.learned_grad(p, x, t)
    want = ref.grad(p.astype(np.float64), x, t)
    # sums of up to 128 products rounded at 2^-24 each, inputs of order one
    assert np.abs(g - want).max() <= 1e-3 * np.abs(want).max() + 1e-6
    assert abs(loss - ref.loss(p.astype(np.float64), x, t)) <= 1e-4 * (1 + loss)


def fma(a, b, c):
    """Fused multiply-add in binary32 (but for a tie of the binary64 sum)."""
    return (a.astype(np.float64) * b.astype(np.float64) + c).astype(np.float32)


def train32(xs, ts, steps):
    """The training loop in binary32: every sum in index order, fused."""
    f = np.float32
    h = ref.H
    s = len(xs)
    q = xs[np.minimum(np.arange(h + 1) * s // h, s - 1)]
    span = np.maximum(q[1:] - q[:-1], f(2.0 ** -24))
    p = np.concatenate([f(1) / span, -q[:-1] / span, np.eye(h, dtype=f).ravel(), np.zeros(h, f),
                        np.full(h, f(1) / f(h)), np.zeros(1, f)]).astype(f)
    nonneg = np.zeros(ref.NPARAM, bool)
    nonneg[:h] = nonneg[2 * h:2 * h + h * h] = nonneg[3 * h + h * h:-1] = True
    m, v = np.zeros_like(p), np.zeros_like(p)
    b1, b2, lr, eps, one = f(0.9), f(0.999), f(1e-3), f(1e-8), f(1)
    b1t, b2t = one, one
    clip = lambda a: np.minimum(np.maximum(a, f(0)), one)
    inside = lambda a: ((a > 0) & (a < 1)).astype(f)
    for st in range(steps):
        pick = [(st * 128 + i) * 2654435761 % s for i in range(128)]
        x, t = xs[pick], ts[pick]
        w1, c1 = p[:h], p[h:2 * h]
        W2 = p[2 * h:2 * h + h * h].reshape(h, h)
        c2, w3, c3 = p[2 * h + h * h:3 * h + h * h], p[3 * h + h * h:-1], p[-1]
        a1 = fma(np.broadcast_to(w1, (128, h)), x[:, None], c1)
        h1 = clip(a1)
        a2 = np.broadcast_to(c2, (128, h)).astype(f)
        for j in range(h):
            a2 = fma(W2[None, :, j], h1[:, j, None], a2)
        h2 = clip(a2)
        y = np.full(128, c3, f)
        for i in range(h):
            y = fma(w3[i], h2[:, i], y)
        g = f(2) * (y - t) / f(128)
        d2 = g[:, None] * w3 * inside(a2)
        e3 = g[:, None] * h2
        d1 = np.zeros((128, h), f)
        for i in range(h):
            d1 = fma(d2[:, i, None], W2[None, i, :], d1)
        d1 = d1 * inside(a1)
        d1x = d1 * x[:, None]
        gW, gb2, gw3 = np.zeros((h, h), f), np.zeros(h, f), np.zeros(h, f)
        gw1, gb1, gb3 = np.zeros(h, f), np.zeros(h, f), f(0)
        for b in range(128):
            gW = fma(d2[b, :, None], h1[b, None, :], gW)
            gb2, gw3, gw1, gb1, gb3 = (gb2 + d2[b], gw3 + e3[b], gw1 + d1x[b], gb1 + d1[b],
                                       gb3 + g[b])
        grad = np.concatenate([gw1, gb1, gW.ravel(), gb2, gw3, [gb3]]).astype(f)
        b1t, b2t = b1t * b1, b2t * b2
        m = b1 * m + (one - b1) * grad
        v = b2 * v + (one - b2) * grad * grad
        p = p - lr * (m / (one - b1t)) / (np.sqrt(v / (one - b2t)) + eps)
        p[nonneg] = np.maximum(p[nonneg], f(0))
    return p


@pytest.mark.parametrize("n,steps", [(2, 3), (100, 0), (100, 1), (5000, 20), (100_000, 64)])
def test_training_is_the_plain_loop(n, steps):
    pts = workload.uniform_points(n, 77)
    idx = sfc.Index(torch.as_tensor(pts).to("cuda:0"), sfc.MORTON)
    idx.learned_fit(steps)
    p = idx.learned_params()
    keys = np.sort(oracle.keys(pts, sfc.MORTON))
    s = 1 << 16
    while s > n:
        s >>= 1
    at = np.arange(s) * n // s
    xs = ((keys[at] >> np.uint64(40)).astype(np.float64) / 2.0 ** 24).astype(np.float32)
    want = train32(xs, (at / n).astype(np.float32), steps)
    # the same roundings, but for a rare tie in the binary64 sums above
    assert np.linalg.norm(p - want) <= 1e-6 * np.linalg.norm(want)
    idx.close()
