"""The attraction of rows so long that a chunk holds a few of them, more chunks
than 32 rows a chunk would make: the same bits for every split of the work over
blocks, and row sums against those of all pairs in FP64 (1e-4 in FP32, 1e-10 in FP64).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _dense(n, per, seed):
    rng = np.random.default_rng(seed)
    P = np.zeros((n, n))
    for i in range(n):
        j = rng.choice(n - 1, per, replace=False)
        P[i, j + (j >= i)] = rng.random(per)
    P /= P.sum()
    row, col = np.nonzero(P)
    rp = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
    return P, (rp, col.astype(np.int32), P[row, col])


@pytest.mark.parametrize("prec,tol", [(0, 1e-4), (1, 1e-10)])
@pytest.mark.parametrize("n,per", [(700, 699), (1500, 600)])
def test_dense_rows(n, per, prec, tol):
    from paper_1611_02568_amd import pixelsne
    P, csr = _dense(n, per, n)
    z = np.random.default_rng(1).random((n, 2)) * 255.0
    s = np.array([0.2, 0.3])
    states = []
    for side, helper, fork in [(2, 3, 0), (2, 3, 1), (1, 0, 1), (0, 3, 2), (16, 16, 1)]:
        ctx = pixelsne.Context.from_P(*csr, screen=256, precision=prec, attract_blocks_per_cu=side,
                                      attract_help_blocks_per_cu=helper, attract_fork=fork)
        zt = torch.as_tensor(z).to(ctx.state_dtype)
        ctx.set_state(zt, s, iteration=1000)
        if not states:
            A = ctx.gradient()["A"].double().cpu().numpy()
            zz = zt.double().numpy()
            d = zz[:, None] - zz[None]
            w = P / (1.0 + ((d * s) ** 2).sum(2))
            want = (w[:, :, None] * d).sum(1)
            assert np.linalg.norm(A - want) <= tol * np.linalg.norm(want)
            ctx.set_state(zt, s, iteration=1000)
        ctx.step(6)
        states.append(ctx.get_state())
    for st in states[1:]:
        for key in ("z", "u", "g"):
            assert torch.equal(st[key], states[0][key]), key
