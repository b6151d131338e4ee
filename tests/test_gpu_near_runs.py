"""The embedding's 2-D neighbours of more points than one launch takes (2^20):
points of both launches, the first and last of each among them, against the
squared distances to all points (as in the tests at the edges of the tiles).
"""
import numpy as np
import pytest
import torch

from paper_1611_02568_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
def test_points_of_both_launches(prec):
    from paper_1611_02568_amd import pixelsne
    n, r = (1 << 20) + 131, 1024
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1)
    ctx = pixelsne.Context.from_P(rp, np.sort(col, 1).ravel().astype(np.int32),
                                  np.full(2 * n, 1.0 / (2 * n)), screen=r, precision=prec)
    z = datagen.uniform_pixels(n, r, seed=n, dtype=np.float64 if prec else np.float32)
    s = (0.25, 0.5)
    ctx.set_state(torch.as_tensor(z), s)
    lo = ctx.knn2d().cpu().numpy()
    assert lo.min() >= 0 and lo.max() < n
    y = z.astype(np.float64) * np.array(s)
    # the order of the launches is the Morton order: its ends and its middle
    px = z.astype(np.int64)
    key = sum(((px[:, a] >> b) & 1) << (2 * b + a) for a in (0, 1) for b in range(10))
    order = np.argsort(key, kind="stable")
    rows = np.concatenate([order[:8], order[(1 << 20) - 8:(1 << 20) + 8], order[-8:],
                           np.random.default_rng(1).choice(n, 40, replace=False)])
    for i in rows:
        d = (y[:, 0] - y[i, 0]) ** 2 + (y[:, 1] - y[i, 1]) ** 2
        d[i] = np.inf
        assert len(set(lo[i].tolist())) == 32 and i not in lo[i]
        want = np.sort(np.partition(d, 32)[:32])
        np.testing.assert_allclose(d[lo[i]], want, rtol=4 * 2.0 ** -53, atol=0)
