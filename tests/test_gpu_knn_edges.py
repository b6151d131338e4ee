"""Exact kNN at the edges of its tiles, depth stages, lists and number ranges.

Against the CPU oracle: indices exact (ties to the smaller index), FP64
distances to 1e-13 relative, as in the setup parity tests.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _check(X, k):
    from paper_1611_02568_amd import pixelsne
    idx, d2 = pixelsne.knn(torch.as_tensor(X).cuda(), k)
    oi, od = oracle.knn(X.astype(np.float64), k)
    assert np.array_equal(idx.cpu().numpy(), oi)
    np.testing.assert_allclose(d2.cpu().numpy(), od, rtol=1e-13, atol=0)


def _data(n, D, dtype, seed):
    rng = np.random.default_rng(seed)
    if dtype == np.uint8:
        return rng.integers(0, 256, (n, D), dtype=np.uint8)
    return (3.0 * rng.standard_normal((4, D))[rng.integers(0, 4, n)]
            + rng.standard_normal((n, D))).astype(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64, np.uint8])
@pytest.mark.parametrize("n,k", [(2, 1), (33, 32), (127, 5), (129, 128), (255, 222), (256, 223),
                                 (257, 224), (385, 256), (513, 100), (1025, 256)])
def test_row_edges(n, k, dtype):
    _check(_data(n, 20, dtype, n), k)


@pytest.mark.parametrize("dtype", [np.float32, np.uint8])
@pytest.mark.parametrize("D", [1, 15, 16, 17, 31, 32, 33, 63, 64, 127, 128, 129, 160, 255, 256,
                               257, 784, 1000])
def test_depth_edges(D, dtype):
    _check(_data(700, D, dtype, D), 20)


@pytest.mark.parametrize("dtype", [np.float32, np.uint8])
def test_lists_that_fill_with_ties(dtype):
    """Every point 40 times: whole tiles at one distance, ties cut by index."""
    X = np.repeat(_data(60, 12, dtype, 1), 40, axis=0)
    X = X[np.random.default_rng(2).permutation(len(X))]
    _check(X, 60)


def test_many_rows_cut_lists():
    _check(_data(9000, 24, np.float32, 7), 150)


@pytest.mark.parametrize("scale", [1e-18, 1e-6, 1e6, 1e17])
def test_number_ranges(scale):
    """Far from 1 the halves are scaled by a power of two."""
    _check((_data(400, 40, np.float64, 3) * scale).astype(np.float32), 30)


def test_outliers_and_small_entries():
    """A few rows a thousand times longer than the rest, and columns a
    thousand times smaller: rows the pre-selection cannot prove are recomputed."""
    X = _data(600, 30, np.float32, 4)
    X[::97] *= 1000.0
    X[:, ::3] *= 1e-3
    _check(X, 25)
