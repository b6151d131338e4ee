"""Approximate kNN of rows that hold NaN: every list entry is a row of the data,
once, in order of (squared distance, index) with distances that are no number
behind all others, by index.

One leaf of all rows: the lists are those of a sort over all pairs (indices
equal, distances to 1e-14; a few rows with NaN, so many that lists must name
some, all but one).  Several trees and rounds: indices in range and distinct,
distances those of the pairs, in order.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rows(n, D, bad, x, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, D)).astype(np.float32 if x == "f32" else np.float64)
    rows = rng.choice(n, bad, replace=False)
    X[rows, rng.integers(0, D, bad)] = np.nan
    return X


def _run(X, k, **kw):
    from paper_1611_02568_amd import pixelsne
    idx, d2 = pixelsne.knn_approx(torch.as_tensor(X).cuda(), k, seed=5, **kw)
    return idx.cpu().numpy(), d2.cpu().numpy()


@pytest.mark.parametrize("x", ["f32", "f64"])
@pytest.mark.parametrize("n,D,k,bad,explore", [(40, 5, 30, 20, 1), (300, 7, 256, 100, 0),
                                               (300, 7, 256, 299, 1), (1200, 17, 20, 3, 1),
                                               (1200, 17, 90, 1195, 1), (9000, 4, 10, 4500, 0)])
def test_one_leaf(x, n, D, k, bad, explore):
    X = _rows(n, D, bad, x, n + k)
    idx, d2 = _run(X, k, trees=1, leaf_size=max(n, 2 * k + 2), explore=explore)
    X64 = X.astype(np.float64)
    for i in np.random.default_rng(0).choice(n, min(n, 60), replace=False):
        d = ((X64 - X64[i]) ** 2).sum(1)
        order = np.lexsort((np.arange(n), np.where(np.isnan(d), 0.0, d), np.isnan(d)))
        want = order[order != i][:k]
        assert np.array_equal(idx[i], want)
        np.testing.assert_allclose(d2[i], d[want], rtol=1e-14, atol=0, equal_nan=True)


@pytest.mark.parametrize("x", ["f32", "f64"])
@pytest.mark.parametrize("bad", [250, 4000])
def test_trees(x, bad):
    n, k = 5000, 12
    X = _rows(n, 8, bad, x, bad)
    idx, d2 = _run(X, k, trees=3, explore=2)
    assert idx.min() >= 0 and idx.max() < n
    assert not np.any(idx == np.arange(n)[:, None])
    assert all(len(set(row)) == k for row in idx.tolist())
    X64 = X.astype(np.float64)
    np.testing.assert_allclose(d2, ((X64[:, None] - X64[idx]) ** 2).sum(2), rtol=1e-14, atol=0,
                               equal_nan=True)
    key = np.where(np.isnan(d2), np.inf, d2)
    a, b = key[:, :-1], key[:, 1:]
    assert np.all((a < b) | ((a == b) & (idx[:, :-1] < idx[:, 1:])))
