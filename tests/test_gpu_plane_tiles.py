"""The humans' planar field by tiles, at its edges: planes a pixel short of
or past a tile (64 columns x 8 rows per wave, 32 per workgroup), disks partly
or wholly outside, discs of the most rows its coverage words reach and one
more, crowds whose discs join (runs of covered pixels longer than the words,
depths beyond their rows), discs that cover the plane, and as many chords as
the tiled kernel takes and one more.  A grid of two layers shows every planar
value on both sides; the int32 result is unique and compared exactly."""
import numpy as np
import pytest

import oracle
import scenegen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H = 0.02


def check(dev, nx, ny, xy, radius, nz=2):
    import paper_2201_05058_amd as pc
    g = scenegen.Grid(nx, ny, nz, H)
    print(f"planes {nx}x{ny} n={xy.shape[0]} K={xy.shape[1]} r={radius}",
          flush=True)
    occ = np.zeros(g.shape_zyx, np.uint8)  # an empty room: the humans alone
    rs, _ = oracle.build_static(g, occ)
    wc, _ = oracle.predicted_composite(g, rs, xy, radius, H)
    c, _ = pc.predicted_composite_sdf(g, torch.from_numpy(rs).to(dev), xy,
                                      radius, H, want_sdf=False)
    np.testing.assert_array_equal(c.cpu().numpy(), wc)


@pytest.mark.parametrize("nx,ny", [(1, 1), (63, 31), (64, 32), (65, 33),
                                   (129, 7), (128, 9), (20, 200), (300, 40)])
@pytest.mark.parametrize("r", [0.0, 0.3, 5.0, 12.5])  # pixels
def test_tile_edges(dev, nx, ny, r):
    rng = np.random.default_rng(nx * ny)
    xy = rng.uniform(-1.2 * r - 1, 1.2 * r + 1, size=(3, 3, 2))
    xy += rng.uniform(0, 1, size=(3, 3, 2)) * [nx, ny]
    check(dev, nx, ny, xy * H, r * H)


@pytest.mark.parametrize("r", [27.4, 27.6, 28.4, 60.0, 400.0])
def test_large_discs(dev, r):
    rng = np.random.default_rng(int(10 * r))
    check(dev, 200, 150, rng.uniform(0, 180, size=(2, 2, 2)) * H, r * H)


@pytest.mark.parametrize("k,spread", [(8, 30.0), (16, 90.0), (60, 60.0),
                                      (61, 90.0), (60, 300.0)])
def test_crowds(dev, k, spread):
    # 13 pixels: 27 rows; 61 discs are the most the tiles take
    rng = np.random.default_rng(k)
    xy = 100 + rng.uniform(-spread / 2, spread / 2, size=(2, k, 2))
    xy[1] = xy[0, :1] + np.arange(k)[:, None] * [9.0, 0.5] - [60, 0]  # a chain
    check(dev, 330, 180, xy * H, 13.0 * H)


def test_batch_of_crowds(dev):
    import paper_2201_05058_amd as pc
    rng = np.random.default_rng(5)
    scenes, want = [], []
    for nx, ny, k, r in [(130, 66, 3, 5.0), (200, 150, 2, 40.0),
                         (190, 100, 40, 13.0), (64, 64, 0, 5.0)]:
        g = scenegen.Grid(nx, ny, 2, H)
        xy = rng.uniform(0, 100, size=(2, k, 2)) * H
        rs, _ = oracle.build_static(g, np.zeros(g.shape_zyx, np.uint8))
        want.append(oracle.predicted_composite(g, rs, xy, r * H, H)[0])
        scenes.append({"grid": g, "static_ssq": torch.from_numpy(rs).to(dev),
                       "human_xy": xy, "radius": r * H, "height": H,
                       "want_sdf": False})
    for (c, _), w in zip(pc.predicted_composite_sdf_batch(scenes), want):
        np.testing.assert_array_equal(c.cpu().numpy(), w)
