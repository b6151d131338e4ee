"""The embedding's 2-D neighbours and its KL at the edges of their tiles.

Neighbours: tiles of 64 points, groups of 64 tiles, a list of 32; many points
on one spot, in one pixel, or spread so that every box matters.  KL: tiles of
256 points, an odd and an even number of them.
"""
import numpy as np
import pytest
import torch

from paper_1611_02568_amd import datagen

pytestmark = pytest.mark.gpu


def _ring_P(n):
    if n == 2:
        return np.array([0, 1, 2], np.int64), np.array([1, 0], np.int32), np.array([0.5, 0.5])
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1)
    return rp, np.sort(col, 1).ravel().astype(np.int32), np.full(2 * n, 1.0 / (2 * n))


def _positions(kind, n, r, dtype):
    if kind == "uniform":
        return datagen.uniform_pixels(n, r, seed=n, dtype=dtype)
    z = datagen.clustered_pixels(n, r, seed=n, spread=0.001, dtype=dtype)
    if kind == "one_spot":
        z[: n // 2] = z[5]
    return z


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind", ["uniform", "clustered", "one_spot"])
@pytest.mark.parametrize("n", [33, 64, 65, 129, 4096, 4097])
def test_neighbours_at_tile_edges(n, kind, prec):
    from paper_1611_02568_amd import pixelsne
    r = 64
    z = _positions(kind, n, r, np.float64 if prec else np.float32)
    ctx = pixelsne.Context.from_P(*_ring_P(n), screen=r, precision=prec)
    s = (0.25, 0.5)                       # powers of two: the metric is exact up to its sums
    ctx.set_state(torch.as_tensor(z), s)
    lo = ctx.knn2d().cpu().numpy()
    y = z.astype(np.float64) * np.array(s)
    for i in np.unique(np.linspace(0, n - 1, 64).astype(int)):
        d = (y[:, 0] - y[i, 0]) ** 2 + (y[:, 1] - y[i, 1]) ** 2
        d[i] = np.inf
        assert len(set(lo[i].tolist())) == 32 and i not in lo[i]
        want = np.sort(d)[:32]
        # the two sides round the same sum of two squares once differently
        np.testing.assert_allclose(d[lo[i]], want, rtol=4 * 2.0 ** -53, atol=0)
        same = d[lo[i]][1:] == d[lo[i]][:-1]
        assert np.all(lo[i][1:][same] > lo[i][:-1][same])      # exact ties: smaller index first


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [2, 255, 256, 257, 512, 513, 1025, 1300])
def test_kl_at_tile_edges(n, prec):
    from paper_1611_02568_amd import pixelsne
    z = _positions("clustered" if n > 2 else "uniform", n, 64, np.float64 if prec else np.float32)
    rp, col, val = _ring_P(n)
    ctx = pixelsne.Context.from_P(rp, col, val, screen=64, precision=prec)
    s = np.array([0.3, 0.2])
    ctx.set_state(torch.as_tensor(z), s)
    y = z.astype(np.float64) * s
    d = ((y[:, None, :] - y[None, :, :]) ** 2).sum(2)
    Z = (1.0 / (1.0 + d)).sum() - n
    row = np.repeat(np.arange(n), np.diff(rp))
    want = (val * (np.log(val) + np.log(1.0 + d[row, col]))).sum() + val.sum() * np.log(Z)
    # FP32 terms (a few roundings each) summed in FP32 over at most 256: at
    # most 260 roundings of 2^-24 on Z; P rounded to FP32 once
    assert abs(ctx.kl() - want) <= 260 * 2.0 ** -24 + 1e-6
    assert ctx.kl_noalloc() == ctx.kl()
