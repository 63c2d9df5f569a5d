"""The mesh hierarchy does not depend on whether threads build it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_05581_amd", "csrc")


def _lines(tmp_path, name, threshold, args, flags):
    exe = os.path.join(tmp_path, name)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *flags,
                    f"-DMSK_BVH_THREAD_ELEMS={threshold}", "-pthread", "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "bvh_driver.cpp"), os.path.join(CSRC, "bvh_build.cpp")],
                   check=True, timeout=300)
    out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=300)
    return out.stdout.splitlines()


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("flags", [("-O2",), ("-O1", "-g", "-fsanitize=thread")], ids=["plain", "threads_checked"])
def test_threads_build_the_same_tree(tmp_path, flags):
    """Sizes about n / 16 elements per range, every leaf width, an axis without extent, coincident centroids and
    a crowded bin: the same nodes and leaf order, byte for byte."""
    args = []
    for n in (1, 2, 15, 16, 17, 33, 257, 4096, 8193):
        for leaf in (1, 4, 8):
            for kind in (0, 1, 2, 3):
                args += [n, leaf, kind]
    serial = _lines(tmp_path, "serial", 1 << 30, args, flags)
    threaded = _lines(tmp_path, "threaded", 1, args, flags)
    assert len(serial) == len(args) // 3
    assert serial == threaded
