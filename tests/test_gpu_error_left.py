"""A call that finds no memory says so by its status and leaves no HIP error
behind for the program's next GPU call to trip over.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _network(pixelsne):
    net = pixelsne.MLP(4, 30000, 2)            # 2^20 rows: 400 GB of activations
    try:
        net.grad(torch.zeros(1 << 20, 4, device="cuda"), torch.zeros(1 << 20, 2, device="cuda"))
    finally:
        net.close()


def _knn(pixelsne):
    # lists as large as the outputs, of which the device holds one
    pixelsne.knn_approx(torch.zeros(300_000_000, 1, dtype=torch.uint8, device="cuda"), 60, trees=1,
                        explore=0)


@pytest.mark.parametrize("call", [_network, _knn])
def test_no_error_left(call):
    from paper_1611_02568_amd import pixelsne
    torch.cuda.empty_cache()
    with pytest.raises(pixelsne.PixelSNEError, match="out of device memory"):
        call(pixelsne)
    torch.cuda.empty_cache()
    assert float(torch.ones(1000, device="cuda").add_(1.0).sum()) == 2000.0
