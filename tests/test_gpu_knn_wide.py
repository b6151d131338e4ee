"""Exact kNN of rows so many and so long that packing them takes more than one
launch (2^26 pieces of 16 bytes): lists of sampled rows, from all over the data,
against distances to every row (whole numbers for bytes; FP64 else, 1e-12).
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x,n,D", [("u8", 36000, 32000), ("f32", 290000, 2000)])
def test_rows_of_every_launch(x, n, D):
    from paper_1611_02568_amd import pixelsne
    k = 20
    g = torch.Generator(device="cuda").manual_seed(D)
    if x == "u8":
        X = torch.randint(0, 256, (n, D), device="cuda", generator=g, dtype=torch.uint8)
    else:
        X = torch.randn(n, D, device="cuda", generator=g)
    idx, d2 = pixelsne.knn(X, k)
    rows = torch.cat([torch.arange(3, device="cuda"), torch.arange(n - 3, n, device="cuda"),
                      torch.randint(0, n, (14,), device="cuda", generator=g)])
    for i in rows.tolist():
        d = torch.empty(n, dtype=torch.float64, device="cuda")
        for a in range(0, n, 2000):
            e = X[a:a + 2000].double() - X[i].double()
            d[a:a + 2000] = (e * e).sum(1)
        d[i] = float("inf")
        want, at = d.sort(stable=True)
        torch.testing.assert_close(d2[i], want[:k], rtol=0 if x == "u8" else 1e-12, atol=0)
        assert torch.equal(idx[i].long(), at[:k])
