"""The network's forward pass where the free memory has no room for a whole pass
of 32,768 rows: outputs equal to those with all memory free, also afterwards.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

MB = 1 << 20


def test_short_of_memory():
    from paper_1611_02568_amd import pixelsne
    n, d = 40000, 20000
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(n, d, device="cuda", generator=g)
    nets = [pixelsne.MLP(d, 16, 16, seed=1) for _ in range(2)]
    nets[1].set_params(nets[0].params())
    want = nets[0].forward(X)
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    rest = []
    try:
        while (left := torch.cuda.mem_get_info()[0] - 600 * MB) > 2 * MB:
            rest.append(torch.empty(min(left, 1 << 34), dtype=torch.uint8, device="cuda"))
        L = pixelsne.load()
        rc = L.pixelsne_mlp_forward(nets[1]._h, pixelsne._ptr(X), n, pixelsne._ptr(out))
    finally:
        del rest
        torch.cuda.empty_cache()
    assert rc == 0, L.pixelsne_last_error()
    assert torch.equal(out, want)
    assert torch.equal(nets[1].forward(X), want)
