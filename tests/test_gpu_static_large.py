"""Static builds of 3 2^24 voxels and more, against the oracle, bit for bit
(the results are whole numbers, and the fp32 field the same correctly rounded
root and product of them).

Such a build looks whether every voxel has one of the other type near
(within 169 voxels, bounded from blocks of 16) and then propagates along the
columns in 16 bits; else it takes the envelopes.  Shapes: the three widths of
the x pass's packs (256, 512, 880 voxels), columns of 512, a few and one rows
past a wave's 32, tiles of fewer than 128 columns.  Contents: boxes (near,
with deep insides), walls of one voxel's thickness, dense and thin noise and
dust (near, with distances up to the limit), one voxel of either kind, none,
all (not near).
"""
import numpy as np
import pytest

import oracle
import scenegen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(512, 448, 256), (229, 505, 512), (223, 300, 880)]  # nz, ny, nx


def contents(shape, rng):
    box = np.zeros(shape, np.uint8)
    for _ in range(60):
        b = [int(rng.integers(8, 90)) for _ in shape]
        a = [int(rng.integers(0, max(1, n - s))) for n, s in zip(shape, b)]
        box[a[0]:a[0] + b[0], a[1]:a[1] + b[1], a[2]:a[2] + b[2]] = 1
    yield "boxes", box
    wall = np.zeros(shape, np.uint8)
    wall[::127] = 1
    wall[:, 200] = 1
    wall[:, 17:, 100] = 1
    yield "walls", wall
    yield "thin noise", (rng.random(shape, np.float32) < 2e-5).astype(np.uint8)
    yield "dust", (rng.random(shape, np.float32) < 4e-6).astype(np.uint8)
    yield "dense noise", (rng.random(shape, np.float32) < 0.7).astype(np.uint8)
    one = np.zeros(shape, np.uint8)
    one[-1, 3, 0] = 1
    yield "one occupied", one
    yield "one free", 1 - one
    yield "none", np.zeros(shape, np.uint8)
    yield "all", np.ones(shape, np.uint8)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_large_static_build_matches_oracle(dev, shape):
    import paper_2201_05058_amd as pc
    assert np.prod(shape, dtype=np.int64) >= 3 << 24
    rng = np.random.default_rng(sum(shape))
    grid = scenegen.Grid(shape[2], shape[1], shape[0], 0.05)
    ssq = torch.empty(shape, dtype=torch.int32, device=dev)
    sdf = torch.empty(shape, device=dev)
    for name, occ in contents(shape, rng):
        print(f"large static shape={shape} {name}", flush=True)
        rs, rf = oracle.build_static(grid, occ)
        rs, rf = torch.from_numpy(rs).to(dev), torch.from_numpy(rf).to(dev)
        occ_d = torch.from_numpy(occ).to(dev)
        for want_sdf in (True, False):
            ssq.zero_()
            sdf.fill_(-7.0)
            pc.build_static_sdf(grid, occ_d, ssq=ssq,
                                sdf=sdf if want_sdf else None,
                                want_sdf=want_sdf)
            assert torch.equal(ssq, rs), name
            assert not want_sdf or torch.equal(sdf, rf), name
