"""Surrogate queries among many humans: up to 32 a query's relevant humans are
the bits of one word, beyond they are found again by each kernel.  Same
comparison and bounds as the other surrogate queries."""
import pytest

from test_gpu_surrogate import test_queries_match_oracle as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("humans", [31, 32, 33, 45])
def test_many_humans(dev, humans):
    import paper_2201_05058_amd.surrogate as sg
    # seed, Q, nx, ny, nz, slices, humans, voxel, boxes, margin, band
    check(sg, dev, (40 + humans, 2500, 90, 80, 24, 3, humans, 0.08, 4, 0.02,
                    0.05))
