"""Composites of grids beyond the caches, whose launch shape and 16-bit static
copy depend on the grid's size, the fields and the number of slices: the
default's outputs equal those of single slices read from the field itself
(the shape the oracle's tests cover), on both sides of each line."""
import numpy as np
import pytest

import scenegen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nz,ny,nx,n", [
    (119, 512, 512, 11), (120, 512, 512, 11), (239, 512, 512, 5),
    (240, 512, 512, 16), (240, 512, 512, 15), (256, 512, 512, 17),
    (256, 512, 512, 4), (257, 512, 512, 8), (257, 512, 512, 6),
    (300, 509, 511, 7), (320, 512, 512, 9), (321, 512, 512, 13),
    (321, 512, 512, 3), (263, 541, 601, 5)])
def test_default_shape_equals_single_slices(dev, nz, ny, nx, n):
    import paper_2201_05058_amd as pc
    g = scenegen.Grid(nx, ny, nz, 0.01)
    rng = np.random.default_rng(nz + n)
    occ = torch.zeros(g.shape_zyx, dtype=torch.uint8, device=dev)
    for _ in range(6):
        a = [int(rng.integers(0, s - 40)) for s in g.shape_zyx]
        occ[a[0]:a[0] + 30, a[1]:a[1] + 40, a[2]:a[2] + 35] = 1
    s, _ = pc.build_static_sdf(g, occ, want_sdf=False)
    del occ
    xy = rng.uniform(0, 1, size=(n, 3, 2)) * [nx * 0.01, ny * 0.01]
    plain = pc.Handle()
    plain.set_tuning({"composite_slices_per_block": 1, "composite_order": 0,
                      "composite_static16": 1})
    c, f = pc.predicted_composite_sdf(g, s, xy, 0.25, 1.8, handle=plain)
    for want in [(True, True), (True, False), (False, True)]:
        print("composite large", nx, ny, nz, n, want, flush=True)
        got = pc.predicted_composite_sdf(g, s, xy, 0.25, 1.8,
                                         want_ssq=want[0], want_sdf=want[1])
        for a, b, w in zip(got, (c, f), want):
            assert not w or torch.equal(a, b)
        del got
    plain.close()
