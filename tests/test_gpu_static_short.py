"""Static builds with short columns, which propagate in 32 bits, against the
oracle, bit for bit, in grids too long for the 16-bit passes: columns at the
edges of a wave's rows (32, 48, two waves), along y and z, up to the first
that takes the envelopes (64), beside y or z passes of another kind; values
beyond 16 bits (a site hundreds of voxels away).
"""
import numpy as np
import pytest

import oracle
import scenegen
from test_gpu_static_small import contents

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(nz, 140, 190) for nz in (2, 3, 31, 32, 33, 47, 48, 49, 63, 64)]
SHAPES += [(150, ny, 190) for ny in (2, 31, 33, 48, 49, 63, 64)]
SHAPES += [(40, 40, 700), (64, 33, 261), (20, 400, 300)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_short_columns_match_oracle(dev, shape):
    import paper_2201_05058_amd as pc
    rng = np.random.default_rng(sum(shape))
    grid = scenegen.Grid(shape[2], shape[1], shape[0], 0.05)
    for name, occ in contents(shape, rng):
        print(f"short columns shape={shape} {name}", flush=True)
        rs, rf = oracle.build_static(grid, occ)
        occ_d = torch.from_numpy(occ).to(dev)
        ssq = torch.zeros(shape, dtype=torch.int32, device=dev)
        sdf = torch.full(shape, -7.0, device=dev)
        pc.build_static_sdf(grid, occ_d, ssq=ssq, sdf=sdf)
        np.testing.assert_array_equal(ssq.cpu().numpy(), rs)
        np.testing.assert_array_equal(sdf.cpu().numpy(), rf)
        only, _ = pc.build_static_sdf(grid, occ_d, want_sdf=False)
        np.testing.assert_array_equal(only.cpu().numpy(), rs)
