"""The exact kNN of rows that are put in an order first (from 32,768 on, when they
fall into clusters): lists of sampled rows against the oracle's brute force in
FP64, indices equal, squared distances to 1e-12 (whole numbers for bytes).

Cases: clusters smaller than a list, of unequal size and beside each other in a
tile; ties across tiles; an offset and an outlier that widen the error bounds;
rows without structure and all alike, which keep their order; groups of more
than one tile.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _clusters(rng, n, D, sizes, spread):
    lab = np.repeat(np.arange(len(sizes)), sizes)
    lab = np.concatenate([lab, rng.integers(0, len(sizes), n - len(lab))])
    rng.shuffle(lab)
    return spread * rng.standard_normal((len(sizes), D))[lab] + rng.standard_normal((n, D))


@pytest.mark.parametrize("kind,x,n,D,k", [
    ("small", "f32", 32768, 20, 90), ("small", "f64", 32769, 9, 256),
    ("small", "u8", 33001, 24, 60), ("ties", "u8", 33000, 6, 40), ("ties", "f32", 33000, 6, 40),
    ("offset", "f32", 33000, 16, 30), ("outlier", "f32", 33000, 16, 30),
    ("plane", "f32", 40000, 2, 30), ("gauss", "f32", 33000, 8, 30), ("alike", "f32", 33000, 5, 7),
    ("deep", "f32", 33000, 150, 20), ("deep", "u8", 33000, 300, 20),
    ("small", "f32", 1048577 + 300, 3, 5)])
def test_lists(kind, x, n, D, k):
    from paper_1611_02568_amd import pixelsne
    rng = np.random.default_rng(n + D + k)
    sizes = [40, 300, 5, 2000, 700]
    if kind == "small":
        X = _clusters(rng, n, D, sizes, 8.0)
    elif kind == "ties":
        X = np.round(_clusters(rng, n, D, sizes, 20.0))
    elif kind in ("offset", "outlier", "deep"):
        X = _clusters(rng, n, D, [1000] * 12, 6.0)
        if kind == "offset":
            X += 500.0
        if kind == "outlier":
            X[n // 2] = 1e5
    elif kind == "alike":
        X = np.ones((n, D))
    else:
        X = rng.standard_normal((n, D))
    if x == "u8":
        X = np.clip(np.round(X * 5 + 128), 0, 255).astype(np.uint8)
    else:
        X = X.astype(np.float32 if x == "f32" else np.float64)
    idx, d2 = pixelsne.knn(torch.as_tensor(X).cuda(), k)
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    rows = np.unique(np.concatenate([[0, n // 2, n - 1], rng.choice(n, 300, replace=False)]))
    if x == "f32" and kind != "alike":
        # the rows of the smallest cluster: nearest to a row of it
        rows = np.unique(np.concatenate([rows, idx[rows[:20], 0]]))
    oi, od = oracle.knn(X.astype(np.float64), k, rows=rows)
    assert np.array_equal(idx[rows], oi)
    np.testing.assert_allclose(d2[rows], od, rtol=0 if x == "u8" else 1e-12, atol=0)
    # every list ascends by (distance, index) and does not hold its row
    assert np.all(np.diff(d2, axis=1) >= 0)
    assert np.all((np.diff(d2, axis=1) > 0) | (np.diff(idx, axis=1) > 0))
    assert not np.any(idx == np.arange(n)[:, None])
