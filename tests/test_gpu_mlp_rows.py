"""The row-tiled network kernels at the edges of their tiles: 32 rows per
wave, 128 per workgroup, slabs of 32 rows and chunks of the weight gradient,
every input width class (16-byte loads or single ones) and unaligned inputs,
against the fp64 oracle.

Tolerance.  A pre-activation within the fp32 accumulation error of a BF16
rounding boundary may round the other way on the GPU (about one activation
in 1e4).  One such flip moves one activation by up to 2^-8 of itself, hence
the next layer's pre-activations, sums of 128 terms, by about 2^-8 /
sqrt(128) = 3.5e-4 of their RMS; in a batch of a few rows that moves every
value.  So the median is bounded at 2e-3 and the maximum at 5e-2 of the
reference's RMS: a wrong index, a dropped row or a wrong sign moves the
median to order one.
"""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def net_and_rows(dev, seed, n, n_in, shift=0, gain=1.5):
    from paper_2201_05058_amd import surrogate
    r = np.random.default_rng(seed)
    p = omlp.pack([r.uniform(-1, 1, size=s) * gain /
                   np.sqrt(s[-1] if len(s) == 2 else 16)
                   for s in omlp.shapes(n_in)]).astype(np.float32)
    off = (0.1 * r.normal(size=n_in)).astype(np.float32)
    sc = (0.5 + r.random(n_in)).astype(np.float32)
    x = r.normal(size=(n, n_in)).astype(np.float32)
    net = surrogate.Mlp(n_in=n_in)
    net.set_params(p, off, sc, 1.3)
    buf = torch.zeros(n * n_in + shift, device=dev)
    xd = buf[shift:].view(n, n_in)  # 4 * shift bytes past the allocation
    xd.copy_(torch.from_numpy(x))
    return net, p.astype(np.float64), x, xd, (off, sc, 1.3)


def close(got, want, what):
    got = got.cpu().numpy().astype(np.float64).reshape(-1)
    want = np.asarray(want, np.float64).reshape(-1)
    assert np.all(np.isfinite(got)), what
    err = np.abs(got - want) / (np.sqrt(np.mean(want ** 2)) + 1e-30)
    assert np.median(err) <= 2e-3, (what, float(np.median(err)))
    assert err.max() <= 5e-2, (what, float(err.max()))


@pytest.mark.parametrize("n,n_in,shift", [
    (1, 16, 0), (31, 16, 1), (32, 8, 0), (33, 7, 0), (127, 32, 0),
    (128, 17, 3), (129, 24, 0), (1025, 1, 0), (4095, 16, 0), (4129, 16, 2)])
def test_edges_match_oracle(dev, n, n_in, shift):
    net, p, x, xd, nrm = net_and_rows(dev, n + n_in, n, n_in, shift)
    r = np.random.default_rng(n)
    print(f"mlp rows n={n} n_in={n_in} shift={shift}", flush=True)
    wy, _ = omlp.forward(p, x, *nrm)
    y, gx = net.forward(xd)
    close(y, wy, "y")
    close(gx, omlp.input_gradient(p, x, *nrm), "gx")
    assert torch.equal(net.forward(xd, want_grad=False)[0], y)
    dy = r.normal(size=n).astype(np.float32)
    gp, gx = net.gradients(xd, torch.from_numpy(dy).to(dev))
    wg, wgx = omlp.backward(p, x, dy, *nrm)
    for k, (a, b) in enumerate(zip(omlp.unpack(gp.cpu().numpy()),
                                   omlp.unpack(wg))):
        close(torch.from_numpy(a), b, f"parameter {k}")
    close(gx, wgx, "gx of dy")
    t = (wy + r.normal(size=n)).astype(np.float32)
    loss = torch.zeros(1, device=dev)
    gp = net.loss_gradients(xd, torch.from_numpy(t).to(dev), loss)
    wl, wdy = omlp.mse_loss_grad(wy, t)
    wg, _ = omlp.backward(p, x, wdy, *nrm)
    for k, (a, b) in enumerate(zip(omlp.unpack(gp.cpu().numpy()),
                                   omlp.unpack(wg))):
        close(torch.from_numpy(a), b, f"loss parameter {k}")
    assert abs(float(loss) - wl) <= 5e-2 * wl
    net.close()


def test_saturated_units(dev):
    """Pre-activations far beyond |z| = 87, where exp(-z) leaves fp32."""
    net, p, x, xd, nrm = net_and_rows(dev, 3, 200, 16, gain=60.0)
    wy, c = omlp.forward(p, x, *nrm)
    assert max(np.abs(a).max() for a in c["a"]) > 1e3
    y, _ = net.forward(xd)
    close(y, wy, "y")
    dy = np.ones(200, np.float32)
    gp, _ = net.gradients(xd, torch.from_numpy(dy).to(dev))
    wg, _ = omlp.backward(p, x, dy, *nrm)
    for k, (a, b) in enumerate(zip(omlp.unpack(gp.cpu().numpy()),
                                   omlp.unpack(wg))):
        close(torch.from_numpy(a), b, f"parameter {k}")
    net.close()


def test_smaller_batch_after_a_larger_one(dev):
    """The workspace of a larger batch serves a smaller one."""
    net, p, x, xd, nrm = net_and_rows(dev, 11, 5000, 16)
    t = torch.zeros(5000, device=dev)
    first = net.loss_gradients(xd[:300].contiguous(), t[:300])
    net.loss_gradients(xd, t)
    again = net.loss_gradients(xd[:300].contiguous(), t[:300])
    assert torch.equal(first, again)
    net.close()
