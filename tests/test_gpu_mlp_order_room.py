"""Training after a call that found no memory for its order of the rows: the
same weights as a network trains to that never made such a call.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

MB = 1 << 20


def test_training_after_no_memory():
    from paper_1611_02568_amd import pixelsne
    n = 60_000_000
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(n, 1, device="cuda", generator=g)
    Y = torch.rand(n, 2, device="cuda", generator=g)
    nets = [pixelsne.MLP(1, 8, 8, seed=1) for _ in range(2)]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    rest = []
    try:
        while (left := torch.cuda.mem_get_info()[0] - 150 * MB) > 2 * MB:
            rest.append(torch.empty(min(left, 1 << 34), dtype=torch.uint8, device="cuda"))
        with pytest.raises(pixelsne.PixelSNEError, match="memory"):
            nets[0].train(X, Y, 1, batch=1000)
    finally:
        del rest
        torch.cuda.empty_cache()
    X, Y = X[:5000].contiguous(), Y[:5000].contiguous()
    losses = [net.train(X, Y, 2, batch=500) for net in nets]
    assert losses[0] == losses[1]
    assert torch.equal(nets[0].params(), nets[1].params())
