"""Batched composites of one field or both, where an item holds one, two or
four slices: slice counts at the groups' edges, scenes at the sizes where the
rule changes and of one to nine voxel chunks, equal to the plain calls."""
import numpy as np
import pytest

import scenegen
from test_gpu_batch import plain, scene_dict

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DIMS = [(9, 9, 9), (32, 16, 14), (32, 16, 16), (21, 20, 11), (64, 64, 63),
        (64, 64, 64), (65, 63, 65), (130, 70, 33)]


@pytest.mark.parametrize("want", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 9])
def test_fields_and_slices(dev, want, n):
    import paper_2201_05058_amd as pc
    scenes, refs = [], []
    for q, dims in enumerate(DIMS):
        sc = scenegen.small_scene(50 + q, *dims, h=0.05, n_boxes=4,
                                  n_humans=2, n_slices=n)
        d = scene_dict(pc, sc, dev)
        refs.append(plain(pc, d))
        scenes.append({**d, "want_ssq": want[0], "want_sdf": want[1]})
    print("batch fields", want, n, flush=True)
    for got, ref in zip(pc.predicted_composite_sdf_batch(scenes), refs):
        for a, b, w in zip(got, ref, want):
            assert (a is not None) == w
            if w:
                np.testing.assert_array_equal(a.cpu().numpy(),
                                              b.cpu().numpy())
