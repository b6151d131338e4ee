"""Approximate kNN at the edges of its kernels against the oracle, which takes
the same steps in FP64: equal lists, squared distances to 1e-15 (whole numbers
for bytes).

Cases: the smallest and largest k and the smallest n; rows that are no whole
number of 16-byte pieces; both ways of dropping repeated candidates (a bit per
point, a hash set); rows that occur many times; and FP32 data whose squares
overflow or vanish in FP32, where the first look at a distance must say nothing.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psne():
    from paper_1611_02568_amd import pixelsne
    pixelsne.load()
    return pixelsne


@pytest.mark.parametrize("x,n,D,k,trees,explore,scale,repeat", [
    ("f32", 2, 1, 1, 1, 1, 0, 1),
    ("f32", 5, 3, 4, 2, 1, 0, 1),
    ("f64", 300, 3, 7, 2, 2, 0, 1),
    ("f32", 257, 33, 256, 1, 1, 0, 1),
    ("f32", 1500, 17, 256, 2, 1, 0, 1),
    ("f64", 1500, 31, 100, 2, 1, 0, 3),
    ("u8", 2000, 15, 20, 2, 1, 0, 4),
    ("u8", 1025, 31, 64, 3, 1, 0, 1),
    ("f32", 8192, 6, 5, 2, 1, 0, 1),             # a bit per point
    ("f32", 8193, 6, 5, 2, 1, 0, 1),             # the hash set
    ("f32", 9000, 20, 5, 2, 2, 0, 3),
    ("f32", 1200, 20, 20, 2, 1, 80, 1),
    ("f32", 1200, 20, 20, 2, 1, -80, 1),
])
def test_lists(psne, x, n, D, k, trees, explore, scale, repeat):
    rng = np.random.default_rng(n + D + k)
    rows = rng.standard_normal(((n + repeat - 1) // repeat, D))
    X = np.tile(rows, (repeat, 1))[:n]
    if x == "u8":
        X = np.clip(np.round(X * 40 + 128), 0, 255).astype(np.uint8)
    else:
        X = np.ldexp(X.astype(np.float32 if x == "f32" else np.float64), scale)
    idx, d2 = psne.knn_approx(torch.as_tensor(X).cuda(), k, trees=trees, explore=explore, seed=7)
    oi, od = oracle.knn_approx(X.astype(np.float64), k, n_trees=trees, explore=explore, seed=7)
    assert np.array_equal(idx.cpu().numpy(), oi)
    np.testing.assert_allclose(d2.cpu().numpy(), od, rtol=1e-15, atol=0)
