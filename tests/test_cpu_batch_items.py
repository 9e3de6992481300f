"""The batch planner's composite items of scenes of few voxel chunks, on the
CPU: as many chunks as the scene has (up to the next power of two; a multiple
of eight from eight on), and the workers' fields from them equal to the
oracle's.  Chunks of 1024 voxels, one slice per item, counts padded to 64."""
import re
import subprocess

import numpy as np
import pytest

import oracle
import scenegen
from test_cpu_device_code import harness  # noqa: F401  (fixture)


@pytest.mark.parametrize("dims,chunks", [
    ((10, 9, 10), 1), ((20, 9, 11), 2), ((20, 13, 11), 4), ((20, 20, 10), 4),
    ((21, 20, 11), 8), ((20, 20, 20), 8), ((22, 20, 20), 16)])
def test_items_of_small_scenes(harness, tmp_path, dims, chunks):  # noqa: F811
    n = 33
    sc = scenegen.small_scene(sum(dims), *dims, h=0.05, n_boxes=3,
                              n_humans=2, n_slices=n)
    g = sc.grid
    rs, _ = oracle.build_static(g, sc.occ)
    inp, out = str(tmp_path / "b.bin"), str(tmp_path / "b.out")
    with open(inp, "wb") as f:
        f.write(np.array([1, 4, 0, 1, 256, 0], np.int32).tobytes())
        f.write(np.array([*dims, n, 2], np.int32).tobytes())
        f.write(np.array([g.h, *g.origin, sc.radius, sc.height],
                         np.float64).tobytes())
        f.write(np.ascontiguousarray(sc.human_xy, np.float64).tobytes())
        f.write(np.ascontiguousarray(rs, np.int32).tobytes())
    r = subprocess.run([harness, "batch", inp, out], check=True, timeout=120,
                       capture_output=True, text=True)
    items = int(re.search(r"composite items (\d+)", r.stdout).group(1))
    assert items == -(-n * chunks // 64) * 64
    c = np.fromfile(out, dtype=np.int32)[:n * g.nvox]
    wc, _ = oracle.predicted_composite(g, rs, sc.human_xy, sc.radius,
                                       sc.height)
    np.testing.assert_array_equal(c.reshape(wc.shape), wc)
