"""Rows of the exact kNN that the pre-selection's error bound cannot certify: far
from the origin against their distances, all of them (more than one run of
1,024), a few, and with more ties at the k-th distance than one pass collects.
Lists equal to the oracle's in FP64, squared distances to 1e-12.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x", ["f32", "f64"])
@pytest.mark.parametrize("n,D,k,offset,same", [(3000, 64, 20, 3000.0, 0), (257, 33, 256, 1e4, 0),
                                               (1500, 300, 50, 40.0, 0),
                                               (3000, 16, 5, 2000.0, 2500)])
def test_lists(x, n, D, k, offset, same):
    from paper_1611_02568_amd import pixelsne
    rng = np.random.default_rng(n + D)
    X = (offset + rng.standard_normal((n, D))).astype(np.float32 if x == "f32" else np.float64)
    if same:
        X[rng.choice(n, same, replace=False)] = X[0]
    idx, d2 = pixelsne.knn(torch.as_tensor(X).cuda(), k)
    oi, od = oracle.knn(X.astype(np.float64), k)
    assert np.array_equal(idx.cpu().numpy(), oi)
    np.testing.assert_allclose(d2.cpu().numpy(), od, rtol=1e-12, atol=0)
