"""Static builds of grids whose longest distance is at most 169 voxels, which
propagate along the columns in 16 bits whatever the occupancy, against the
oracle, bit for bit (the results are whole numbers, and the fp32 field the
same correctly rounded root and product of them).

Shapes: columns one short of, at and past a wave's 32 rows and their
multiples; passes of two, odd and just over 128 columns; a longest distance
of exactly 169 and one past it (the envelopes).  Each pass has at least
64 tiles of 32 columns, so that none takes the search.  Contents: none, all,
one voxel of either kind, thin walls, thin and dense noise, boxes.
"""
import numpy as np
import pytest

import oracle
import scenegen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(16, ny, 100) for ny in (31, 32, 33, 63, 64, 65, 96, 97, 128)]
SHAPES += [(nz, 16, 100) for nz in (33, 64, 65, 97)]
SHAPES += [(70, 66, 2), (70, 70, 3), (40, 66, 127), (66, 40, 129),
           (25, 64, 64), (64, 64, 64)]
LIMIT = [(64, 97, 125), (64, 97, 126)]


def contents(shape, rng):
    nz, ny, nx = shape
    yield "none", np.zeros(shape, np.uint8)
    yield "all", np.ones(shape, np.uint8)
    one = np.zeros(shape, np.uint8)
    one[-1, -1, 0] = 1
    yield "one occupied", one
    yield "one free", 1 - one
    wall = np.zeros(shape, np.uint8)
    wall[:, ny // 2, : nx // 2] = 1
    wall[nz // 2, :, nx // 3] = 1
    yield "walls", wall
    for p in (0.0003, 0.02, 0.9):
        yield f"noise {p}", (rng.random(shape) < p).astype(np.uint8)
    box = np.zeros(shape, np.uint8)
    for _ in range(3):
        a = [int(rng.integers(0, n)) for n in shape]
        b = [int(rng.integers(1, max(2, n * 2 // 3))) for n in shape]
        box[a[0]:a[0] + b[0], a[1]:a[1] + b[1], a[2]:a[2] + b[2]] = 1
    yield "boxes", box


@pytest.mark.parametrize("shape", SHAPES + LIMIT, ids=str)
@pytest.mark.parametrize("offset", [0, 1])
def test_small_static_build_matches_oracle(dev, shape, offset):
    import paper_2201_05058_amd as pc
    rng = np.random.default_rng(sum(shape))
    grid = scenegen.Grid(shape[2], shape[1], shape[0], 0.05)
    V = int(np.prod(shape))

    def buf(dtype, fill):  # `offset` elements past the allocation's start
        t = torch.full((V + offset,), fill, dtype=dtype, device=dev)
        return t[offset:].view(shape)
    for name, occ in contents(shape, rng):
        print(f"small static shape={shape}+{offset} {name}", flush=True)
        rs, rf = oracle.build_static(grid, occ)
        occ_d = buf(torch.uint8, 0)
        occ_d.copy_(torch.from_numpy(occ))
        ssq, sdf = buf(torch.int32, 0), buf(torch.float32, -7.0)
        pc.build_static_sdf(grid, occ_d, ssq=ssq, sdf=sdf)
        np.testing.assert_array_equal(ssq.cpu().numpy(), rs)
        np.testing.assert_array_equal(sdf.cpu().numpy(), rf)
        only, _ = pc.build_static_sdf(grid, occ_d, want_sdf=False)
        np.testing.assert_array_equal(only.cpu().numpy(), rs)
