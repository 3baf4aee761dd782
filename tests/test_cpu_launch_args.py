"""What the launchers hand to the kernels, on a machine without a GPU: launch_args.cpp,
linked against the library's objects, replaces the kernel launch by a recorder."""
import glob
import os
import subprocess

import pytest

from paper_2602_21203_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    objs = sorted(glob.glob(os.path.join(build.OBJ, "*.o")))
    if len(objs) != len(build.SOURCES):
        pytest.skip("the library's objects are not here (built with it)")
    out = str(tmp_path_factory.mktemp("launch") / "launch_args")
    subprocess.run([build.hipcc(), "-O1", "-std=c++17", f"--offload-arch={build.ARCH}", "-I",
                    os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-x", "hip",
                    os.path.join(HERE, "launch_args.cpp"), "-x", "none", *objs, "-o", out], check=True)
    return out


# adam: the target is a pointer that the kernel may read only where the average has elements.
# ln: the products that normalise their own input refuse buffers that keep no FP32 values,
# and the forms that they are not built for.  tile_lines: from where a product runs on the
# 64 x 64 tile (just above one tile a compute unit it is the slower one).  register_groups:
# where the 32 x 32 tile's groups hold two chunks.  frame_alignment: the update's encoder launch
# reads raw frames at any word, a ring's at any byte.
@pytest.mark.parametrize("check", ["adam_average", "adam_empty_average", "ln_dropped_weights", "ln_dropped_input",
                                   "ln_forms", "tile_lines", "register_groups",
                                   "frame_alignment"])
def test_launch_arguments(program, check):
    assert subprocess.run([program, check], timeout=60).returncode == 0
