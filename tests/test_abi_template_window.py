"""A shifted template's window of more pixels than 32 bits count is refused on
the host, before any device is touched (the address is never dereferenced):
its kernels' pixel numbers would wrap."""
import ctypes as C

import numpy as np
import pytest

import paper_2201_05058_amd as pc
from paper_2201_05058_amd import _native

FAKE = C.c_void_p(0x10000)
ERR_DIMS = 2


# 2 (1024 + 22300 + 2) + 1 and 2 (2 + 30000 + 2) + 1 pixels an axis
@pytest.mark.parametrize("n,radius", [(1024, 22300.0), (2, 30000.0)])
def test_windows_beyond_32_bits_are_refused(n, radius):
    h = pc.Handle()
    g = _native.Grid.make(n, n, 2, 1.0, (0, 0, 0))
    xy = np.zeros((1, 1, 2))
    rc = h.lib.pcsdf_template_composite_sdf(
        h.ptr, C.byref(g), FAKE, 1, 1, xy.ctypes.data_as(C.c_void_p), radius,
        1.8, FAKE, None, None)
    assert rc == ERR_DIMS
    assert "window" in h.lib.pcsdf_last_error(h.ptr).decode()
    h.close()
