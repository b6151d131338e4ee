"""The per-point passes at the edges of their grids (blocks of 256 points, at
most 2,048 of them): after a step the screen scaling spans the screen exactly,
so every block's minimum and maximum took part, and Z is the sum of the
points' Z_i (n non-negative FP64 terms in two orders: n 2^-53 relative).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ring_P(n):
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1)
    return rp, np.sort(col, 1).ravel().astype(np.int32), np.full(2 * n, 1.0 / (2 * n))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [3, 256, 257, 65537, 524288, 524289])
def test_scaling_and_normaliser(n, prec):
    from paper_1611_02568_amd import pixelsne
    r = 256
    rng = np.random.default_rng(n)
    z = (rng.random((n, 2)) * 0.5 + 0.2) * r
    z[-1] = [r - 1.5, 2.5]                      # the extremes lie in the last block
    z[n // 2] = [1.5, r - 2.5]
    ctx = pixelsne.Context.from_P(*_ring_P(n), screen=r, precision=prec)
    ctx.set_state(torch.as_tensor(z.astype(np.float64 if prec else np.float32)),
                  np.array([0.05, 0.06]))
    g = ctx.gradient(1.0)
    zi = g["Zi"].double().cpu().numpy()
    assert abs(g["Z"] - zi.sum()) <= n * 2.0 ** -53 * zi.sum()
    ctx.step(1)
    y = ctx.get_state()["z"].double().cpu().numpy()
    assert np.array_equal(y.min(0), [0.0, 0.0])
    assert np.all(y.max(0) <= r) and np.all(y.max(0) >= r * (1 - 1e-6))
