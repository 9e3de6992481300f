"""The planar field by tiles, with two rows of a column per lane (calls of at
most 192 workgroups of 64 x 32 pixels), four (crowded planes) and eight: the
same planes, disks and crowds on either side of the line, and stacks of planes
so dense that they take the column passes, against the oracle, exactly."""
import numpy as np
import pytest

from test_gpu_plane_tiles import H, check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def slices(nx, ny, many):
    wgs = -(-nx // 64) * -(-ny // 32)
    return 192 // wgs + 1 if many else max(1, min(3, 192 // wgs))


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("nx,ny", [(65, 33), (20, 201), (130, 8), (300, 41)])
@pytest.mark.parametrize("r", [0.3, 5.0, 12.5, 27.4])  # pixels
def test_rows_per_lane(dev, nx, ny, r, many):
    n = slices(nx, ny, many)
    rng = np.random.default_rng(nx + n)
    xy = rng.uniform(-1.2 * r - 1, 1.2 * r + 1, size=(n, 3, 2))
    xy += rng.uniform(0, 1, size=(n, 3, 2)) * [nx, ny]
    check(dev, nx, ny, xy * H, r * H)


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("k,r", [(16, 13.0), (30, 13.0), (4, 27.9)])
def test_crowds_rows_per_lane(dev, k, r, many):
    nx, ny = 230, 140
    n = slices(nx, ny, many)
    rng = np.random.default_rng(k)
    xy = 90 + rng.uniform(-50, 50, size=(n, k, 2))
    xy[0] = xy[0, :1] + np.arange(k)[:, None] * [7.0, 0.5] - [60, 0]
    check(dev, nx, ny, xy * H, r * H)


@pytest.mark.parametrize("ny", [60, 100])
def test_dense_stack(dev, ny):
    # planes covered by their disks, as many as take the column passes
    nx, n = 100, 130
    rng = np.random.default_rng(ny)
    xy = rng.uniform(0, 1, size=(n, 8, 2)) * [nx, ny]
    check(dev, nx, ny, xy * H, 20.4 * H)
