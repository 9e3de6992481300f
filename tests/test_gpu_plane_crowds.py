"""Planar fields of crowds on small planes, on both sides of the line beyond
which they leave the tiles (the boxes' share of the plane times the rows of a
disk), one slice, a few and many; the int32 result is unique and compared
exactly."""
import numpy as np
import pytest

from test_gpu_plane_tiles import H, check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 5, 40])
@pytest.mark.parametrize("nx,ny,k,r", [
    (64, 100, 32, 12.4), (64, 100, 33, 12.4),  # 25 rows: 78.1 and 80.6
    (48, 48, 6, 15.4), (48, 48, 7, 15.4),      # 31 rows: 77.6 and 90.5
    (100, 70, 8, 20.4), (100, 70, 9, 20.4),    # 41 rows: 78.8 and 88.6
    (64, 64, 8, 25.0), (40, 130, 16, 20.0)])
def test_both_sides_of_the_line(dev, nx, ny, k, r, n):
    rng = np.random.default_rng(nx + k)
    xy = rng.uniform(0, 1, size=(n, k, 2)) * [nx, ny]
    xy[0] = 0.5 * np.array([nx, ny]) + 0.2 * (xy[0] - 0.5 * nx)  # joined
    check(dev, nx, ny, xy * H, r * H)
