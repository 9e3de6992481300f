"""What bench.py says of a composite's launch, against the library's rule as
its source states it (no GPU): the 16-bit static copy's limits and the default
shape."""
import os
import re
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(HERE))

import bench  # noqa: E402


def library_constant(path, name):
    with open(path) as f:
        m = re.search(name + r" = (\d+)LL << (\d+);", f.read())
    return int(m.group(1)) << int(m.group(2))


def test_copy_limits_are_the_librarys():
    src = bench.COMPOSITE_SRC
    dev = os.path.join(os.path.dirname(src), "composite_device.h")
    low = library_constant(dev, "kLargeVoxels")
    mid = library_constant(dev, "kSpanVoxels")
    most = library_constant(src, "kCopyVoxels")
    with open(src) as f:
        m = re.search(r"groups >= \(apart \|\| V > kSpanVoxels \? (\d+)"
                      r" : both \? (\d+)",
                      f.read())
    few, many = int(m.group(1)), int(m.group(2))

    def copies(slices, tuning, vox):
        return bench.composite_shape(tuning, vox, slices)[2]
    for v, g in [(low, many), (mid, many), (mid + 1, few), (most, few)]:
        assert copies(g, {}, v) and not copies(g - 1, {}, v)
        t = {"composite_slices_per_block": 3, "composite_order": 1}
        assert copies(3 * g, t, v) and not copies(3 * g - 3, t, v)
    for g3, v3 in [(3, low), (3, mid), (1, low), (1, 1 << 25)]:
        t = {"composite_slices_per_block": g3, "composite_order": 0}
        assert copies(g3 * few, t, v3) and not copies(g3 * (few - 1), t, v3)
        assert not copies(99, t, v3 - 1) or g3 == 1 or v3 == mid
    t = {"composite_slices_per_block": 1, "composite_order": 0}
    assert not copies(99, t, (1 << 25) - 1)
    assert not copies(many, {}, low - 1) and not copies(many, {}, most + 1)
    assert copies(1, {"composite_static16": 2}, 1000)
    assert not copies(2 * many, {"composite_static16": 1}, mid)


def test_launch_shape():
    assert bench.composite_shape({}, 1000, 5)[:2] == (1, 1)
    assert bench.composite_shape({"composite_slices_per_block": 8,
                                  "composite_order": 0}, 1000, 5)[:2] == (5, 0)
    assert bench.composite_shape({"composite_slices_per_block": 2,
                                  "composite_order": 1}, 1000, 5)[:2] == (2, 1)


def test_source_hash_covers_the_kernels_alone(tmp_path):
    """Host-side text of composite.hip leaves the hash as it is, the kernels'
    text and the shared headers' do not."""
    here = os.path.dirname(bench.COMPOSITE_SRC)
    names = ("composite.hip", "composite_device.h", "device_common.h")
    for n in names:
        (tmp_path / n).write_text(open(os.path.join(here, n)).read())
    path = str(tmp_path / "composite.hip")
    h = bench.source_hash(path)
    assert h == bench.source_hash(bench.COMPOSITE_SRC)
    src = (tmp_path / "composite.hip").read_text()
    (tmp_path / "composite.hip").write_text(src + "// host\n")
    assert bench.source_hash(path) == h
    at = src.index("__global__", src.index("k_static16("))
    (tmp_path / "composite.hip").write_text(src[:at] + "/**/" + src[at:])
    assert bench.source_hash(path) != h
    (tmp_path / "composite.hip").write_text(src)
    with open(tmp_path / "device_common.h", "a") as f:
        f.write("// x\n")
    assert bench.source_hash(path) != h
