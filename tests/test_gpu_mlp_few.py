"""Inference on either side of the row count up to which a layer's units are
split over a workgroup's waves: the two kernels do the same operations in the
same order, so a row's value and gradient have the same bits in a batch of any
size; every input width class and unaligned inputs."""
import pytest

from test_gpu_mlp_rows import net_and_rows

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FEW = 32768


@pytest.mark.parametrize("n_in,shift", [(16, 0), (16, 1), (8, 0), (7, 0),
                                        (1, 0), (32, 0), (17, 3)])
def test_same_bits_in_few_and_many_rows(dev, n_in, shift):
    n = FEW + 161  # a remainder of both kernels' tiles
    net, _, _, xd, _ = net_and_rows(dev, n_in + shift, n, n_in, shift)
    print(f"mlp few n_in={n_in} shift={shift}", flush=True)
    y, gx = net.forward(xd)
    assert torch.equal(net.forward(xd, want_grad=False)[0], y)
    for k in (1, 31, 32, 33, 4129, FEW, FEW + 1):
        fy, fg = net.forward(xd[:k])
        assert torch.equal(fy, y[:k]) and torch.equal(fg, gx[:k]), k
        assert torch.equal(net.forward(xd[:k], want_grad=False)[0], fy), k
    net.close()
