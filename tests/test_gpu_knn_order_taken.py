"""Whether the exact kNN takes its rows in cluster order and leaves tiles out, on
inputs that are meant to make it do so or not, and its lists of sampled rows
against the oracle's there: indices equal, squared distances to 1e-12 (whole
numbers for bytes).

Clusters apart; an offset and an outlier that widen the error bound of every
distance, but not beyond what lies between the clusters; an outlier so far away
that the bound says nothing any more; rows without structure, and all alike.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,x,D,taken", [
    ("apart", "f32", 16, True), ("apart", "f64", 16, True), ("apart", "u8", 24, True),
    ("apart", "f32", 150, True), ("apart", "u8", 300, True), ("offset", "f32", 16, True),
    ("outlier", "f32", 16, True), ("outlier", "f64", 40, True), ("far outlier", "f32", 16, False),
    ("gauss", "f32", 16, False), ("gauss", "u8", 16, False), ("alike", "f32", 16, False)])
def test_order(kind, x, D, taken):
    from paper_1611_02568_amd import pixelsne
    n, k = 33001, 30
    rng = np.random.default_rng(D)
    X = rng.standard_normal((n, D))
    if kind not in ("gauss", "alike"):
        X += 8.0 * rng.standard_normal((12, D))[rng.integers(0, 12, n)]
    if kind == "offset":
        X += 200.0
    elif kind.endswith("outlier"):
        X[n // 2] = 300.0 if kind == "outlier" else 1e5
    elif kind == "alike":
        X[:] = 1.0
    if x == "u8":
        X = np.clip(np.round(X * 4 + 128), 0, 255).astype(np.uint8)
    else:
        X = X.astype(np.float32 if x == "f32" else np.float64)
    idx, d2 = pixelsne.knn(torch.as_tensor(X).cuda(), k)
    groups, met, every = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int64()
    pixelsne.load().psne_knn_trace(ctypes.byref(groups), ctypes.byref(met), ctypes.byref(every))
    print(kind, x, D, groups.value, met.value, every.value, flush=True)
    assert every.value == ((n + 127) // 128) * ((n + 255) // 256)
    if taken:
        assert groups.value == (n + 255) // 256
        assert 0 < met.value < every.value // 2
    else:
        assert groups.value == 0
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    rows = np.unique(np.concatenate([[0, n // 2, n - 1], rng.choice(n, 400, replace=False)]))
    oi, od = oracle.knn(X.astype(np.float64), k, rows=rows)
    assert np.array_equal(idx[rows], oi)
    np.testing.assert_allclose(d2[rows], od, rtol=0 if x == "u8" else 1e-12, atol=0)
