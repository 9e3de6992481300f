"""The batch planner's default slices per composite item, on the CPU: one
where both fields of a large scene are written, two in small scenes and four
where one field is written (single slices of one field take up to 1.4 times
as long).  Scenes of whole 1024-voxel chunks; counts padded to 64."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("batch_fields") / "planner")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread",
                    "-I" + os.path.join(HERE, "cpu_device"),
                    "-I" + os.path.join(os.path.dirname(HERE), "include"),
                    "-o", exe, os.path.join(HERE, "cpu_device",
                                            "batch_fields.cpp")], check=True)
    return exe


@pytest.mark.parametrize("dims,n,ssq,sdf,groups", [
    ((64, 64, 64), 21, 1, 1, 21), ((64, 64, 62), 21, 1, 1, 11),
    ((64, 64, 64), 21, 0, 1, 6), ((64, 64, 62), 21, 1, 0, 6),
    ((32, 16, 16), 21, 0, 1, 6), ((32, 16, 14), 21, 1, 0, 11),
    ((32, 16, 14), 21, 1, 1, 11), ((256, 256, 128), 20, 0, 1, 6)])
def test_slices_per_item(planner, dims, n, ssq, sdf, groups):
    chunks = -(-dims[0] * dims[1] * dims[2] // 8192) * 8
    # groups of the largest scene run in spans of ten slices, three groups
    r = subprocess.run([planner, *map(str, (*dims, n, ssq, sdf))],
                       check=True, capture_output=True, text=True, timeout=60)
    assert int(r.stdout) == -(-groups * chunks // 64) * 64
