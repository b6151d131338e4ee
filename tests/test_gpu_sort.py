"""The iteration's key sort at the edges of its tiles and digits: tiles of 2,048
keys up to 262,144 points and of 4,096 above, digits of 1 to 11 bits in one to
three passes.  The exported order is NumPy's stable order of the exported keys,
which are the Morton codes of the pixels.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ring_P(n):
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1)
    return rp, np.sort(col, 1).ravel().astype(np.int32), np.full(2 * n, 1.0 / (2 * n))


def _morton(x, y):
    k = np.zeros(len(x), np.uint64)
    for b in range(16):
        k |= ((x >> b) & 1).astype(np.uint64) << np.uint64(2 * b)
        k |= ((y >> b) & 1).astype(np.uint64) << np.uint64(2 * b + 1)
    return k.astype(np.uint32)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,r", [(3, 2), (63, 4), (2047, 512), (2048, 1024), (2049, 2048),
                                 (5000, 4096), (4097, 65536), (262144, 64), (262145, 2048)])
def test_sorted_order(n, r, prec):
    from paper_1611_02568_amd import pixelsne
    rng = np.random.default_rng(n)
    z = rng.random((n, 2)) ** 2 * r
    z[: n // 3] = z[0]                          # many points in one pixel
    z = np.minimum(z, np.nextafter(np.float32(r), np.float32(0))).astype(
        np.float64 if prec else np.float32)
    ctx = pixelsne.Context.from_P(*_ring_P(n), screen=r, precision=prec)
    ctx.set_state(torch.as_tensor(z), np.array([0.05, 0.06]))
    ctx.gradient(1.0)
    tr = ctx.export_tree()
    keys = tr["keys"].cpu().numpy().view(np.uint32)
    perm = tr["perm"].cpu().numpy()
    px = z.astype(np.float64).astype(np.int64)
    want = _morton(px[:, 0], px[:, 1])
    assert np.array_equal(perm, np.argsort(want, kind="stable"))
    assert np.array_equal(keys, want[perm])
