"""Training gradients where pre-activations are finite and of any size: a
logistic that is merely small, not zero, at z = -87 and beyond would multiply
z into values of order one from |z| = 1e36 on.  Rows whose first layer lies
there contribute as the oracle says, SiLU = SiLU' = 0, beside ordinary rows.
Tolerances are those of the row-tiled kernels' other tests (BF16 rounding
flips), derived there."""
import numpy as np
import pytest

from oracle import mlp as omlp
from test_gpu_mlp_rows import close

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("size", [1e3, 1e30, 1e36, 1e37])
def test_far_negative_units(dev, size):
    from paper_2201_05058_amd import surrogate
    n, n_in = 192, 16
    r = np.random.default_rng(5)
    layers = [r.uniform(-1, 1, size=s) * 1.5 /
              np.sqrt(s[-1] if len(s) == 2 else 16)
              for s in omlp.shapes(n_in)]
    layers[0] = -np.abs(layers[0])  # positive inputs: negative units
    p = omlp.pack(layers).astype(np.float32)
    nrm = (np.zeros(n_in, np.float32), np.ones(n_in, np.float32), 1.3)
    x = r.uniform(0.1, 1.0, size=(n, n_in)).astype(np.float32)
    x[64:] *= np.float32(size)
    net = surrogate.Mlp(n_in=n_in)
    net.set_params(p, *nrm)
    xd = torch.from_numpy(x).to(dev)
    p = p.astype(np.float64)
    print(f"mlp far units size={size}", flush=True)
    wy, _ = omlp.forward(p, x, *nrm)
    close(net.forward(xd)[0], wy, "y")
    dy = r.normal(size=n).astype(np.float32)
    gp, gx = net.gradients(xd, torch.from_numpy(dy).to(dev))
    wg, wgx = omlp.backward(p, x, dy, *nrm)
    for q, (a, b) in enumerate(zip(omlp.unpack(gp.cpu().numpy()),
                                   omlp.unpack(wg))):
        close(torch.from_numpy(a), b, f"parameter {q}")
    close(gx, wgx, "gx")
    net.close()
