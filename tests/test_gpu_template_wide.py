"""Shifted templates whose windows, 2 (nx + m) + 1 pixels wide, exceed a grid's
longest axis (1024): by tiles, by one pixel per lane, and with as many humans
as send narrower windows through the coverage and column passes, which end at
1024 columns.  Humans near x = 0, so that the room's far end reads the
windows' last columns; compared with the oracle's templates exactly."""
import numpy as np
import pytest

import oracle
import scenegen
from oracle.template import template_composite

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H = 0.02


@pytest.mark.parametrize("nx,ny,k,r", [
    (512, 200, 16, 28.3),  # discs of 57 rows, 1085 columns
    (512, 30, 3, 12.0),    # 1053 columns by tiles
    (480, 40, 16, 28.3),   # 1021 columns
    (1010, 24, 8, 5.0),    # 2035 columns by tiles
    (1024, 24, 8, 5.0),    # 2063 columns, past the tiles
    (1024, 24, 2, 5.0)])
def test_wide_windows_match_oracle(dev, nx, ny, k, r):
    import paper_2201_05058_amd as pc
    g = scenegen.Grid(nx, ny, 2, H)
    rng = np.random.default_rng(nx + k)
    xy = np.empty((2, k, 2))
    xy[0] = rng.uniform(0, 1, size=(k, 2)) * [6.0, ny]
    xy[1] = xy[0] + rng.uniform(-2, 2, size=(k, 2))
    rs, _ = oracle.build_static(g, np.zeros(g.shape_zyx, np.uint8))
    print(f"template {nx}x{ny} K={k} r={r}", flush=True)
    c, f = pc.template_composite_sdf(g, torch.from_numpy(rs).to(dev), xy * H,
                                     r * H, H)
    wc, wf = template_composite(g, rs, xy * H, r * H, H)
    np.testing.assert_array_equal(c.cpu().numpy(), wc)
    np.testing.assert_array_equal(f.cpu().numpy(), wf)
