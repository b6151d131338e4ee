"""The FP64 walk where its work split ends: four wavefronts share the walk of 64
points up to 700,000, one walks alone above.  Against the CPU oracle: visits
exact, R and Z within the bars of the gradient parity tests.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_02568_amd import datagen

pytestmark = pytest.mark.gpu


def _ring_P(n):
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1)
    return rp, np.sort(col, 1).ravel().astype(np.int32), np.full(2 * n, 1.0 / (2 * n))


@pytest.mark.parametrize("n", [700000, 700001])
def test_walk_at_the_split_point(n):
    from paper_1611_02568_amd import pixelsne
    r, s = 1024, np.array([0.05, 0.06])
    z = datagen.clustered_pixels(n, r, seed=n, spread=0.05, dtype=np.float64)
    P = _ring_P(n)
    ctx = pixelsne.Context.from_P(*P, screen=r, precision=1, theta=0.5)
    ctx.set_state(torch.as_tensor(z), s)
    g = ctx.gradient(1.0)
    og = oracle.gradient(z, r, s, P, theta=0.5, predicate=0)
    assert np.array_equal(g["visits"].cpu().numpy(), og["visits"])
    R = g["R"].cpu().numpy()
    assert np.linalg.norm(R - og["R"]) <= 1e-10 * np.linalg.norm(og["R"])
    assert abs(g["Z"] - og["Z"]) <= 1e-12 * og["Z"]
