"""Rows that the exact kNN's pre-selection cannot certify, where the free memory
holds its lists but not the scratch of the pass over such rows (25 MB): lists and
distances equal to those found with all memory free.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def most_memory_taken():
    """All but 4 GB of the device's memory held, in pieces, while the module runs."""
    torch.cuda.empty_cache()
    hold = []
    while (left := torch.cuda.mem_get_info()[0] - 4096 * MB) > 2 * MB:
        hold.append(torch.empty(min(left, 1 << 34), dtype=torch.uint8, device="cuda"))
    yield
    del hold
    torch.cuda.empty_cache()


@pytest.mark.parametrize("free", [36, 44])
@pytest.mark.parametrize("same", [0, 2500])
def test_short_of_memory(free, same):
    from paper_1611_02568_amd import pixelsne
    n, D, k = 3000, 64, 20
    rng = np.random.default_rng(n)
    X = 3000.0 + rng.standard_normal((n, D)).astype(np.float32)
    if same:
        X[rng.choice(n, same, replace=False)] = X[0]
    X = torch.as_tensor(X).cuda()
    want, wd = pixelsne.knn(X, k)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    idx, d2 = torch.empty_like(want), torch.empty_like(wd)
    torch.cuda.empty_cache()
    rest = torch.empty(torch.cuda.mem_get_info()[0] - free * MB, dtype=torch.uint8, device="cuda")
    try:
        L = pixelsne.load()
        print("free MB", torch.cuda.mem_get_info()[0] / MB, flush=True)
        rc = L.pixelsne_knn(pixelsne._ptr(X), n, D, pixelsne._X_TYPES[X.dtype], k,
                            pixelsne._ptr(idx), pixelsne._ptr(d2), pixelsne._stream())
    finally:
        del rest
        torch.cuda.empty_cache()
    assert rc == 0, L.pixelsne_last_error()
    assert torch.equal(idx, want) and torch.equal(d2, wd)
