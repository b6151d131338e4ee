"""Exact kNN where device memory is short: less is free than a packed copy of the
rows takes, so that candidates are packed in runs and lists are joined (two to
some fifty runs).  Lists and distances equal to those found with all memory free.
"""
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


def _rows(n, D, x, g):
    lab = torch.randint(0, 9, (n,), device="cuda", generator=g)
    if x == "u8":
        m = torch.randint(40, 200, (9, D), device="cuda", generator=g, dtype=torch.uint8)
        return m[lab] + torch.randint(0, 40, (n, D), device="cuda", generator=g, dtype=torch.uint8)
    dt = torch.float32 if x == "f32" else torch.float64
    m = torch.randn(9, D, device="cuda", generator=g, dtype=dt)
    X = torch.randn(n, D, device="cuda", generator=g, dtype=dt)
    return X.add_(m[lab])


@pytest.mark.parametrize("x,n,D,k,free", [
    ("f32", 5000, 24000, 30, 400), ("f32", 3001, 24000, 256, 140), ("f64", 4100, 16001, 10, 150),
    ("u8", 33000, 8000, 90, 220), ("u8", 2049, 40000, 20, 190), ("f32", 40000, 3000, 40, 350)])
def test_short_of_memory(x, n, D, k, free):
    from paper_1611_02568_amd import pixelsne
    X = _rows(n, D, x, torch.Generator(device="cuda").manual_seed(n))
    want, wd = pixelsne.knn(X, k)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    idx, d2 = torch.empty_like(want), torch.empty_like(wd)
    torch.cuda.empty_cache()
    rest = torch.empty(torch.cuda.mem_get_info()[0] - free * MB, dtype=torch.uint8, device="cuda")
    try:
        L = pixelsne.load()
        rc = L.pixelsne_knn(pixelsne._ptr(X), n, D, pixelsne._X_TYPES[X.dtype], k,
                            pixelsne._ptr(idx), pixelsne._ptr(d2), pixelsne._stream())
        print("free MB", torch.cuda.mem_get_info()[0] // MB, "packed MB",
              n * D * (1 if x == "u8" and D <= 32768 else 4) // MB, flush=True)
    finally:
        del rest
        torch.cuda.empty_cache()
    assert rc == 0, L.pixelsne_last_error()
    assert torch.equal(idx, want) and torch.equal(d2, wd)
