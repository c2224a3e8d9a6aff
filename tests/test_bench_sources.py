"""The benchmark's figures say which kernels they are of (no GPU needed)."""
import glob
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_10247_amd", "csrc")


def test_kernel_hash_covers_every_step_kernel():
    """Every source that defines a step kernel, and every header of ours it includes, is
    hashed: a committed counter summary is not quoted for a kernel that changed since."""
    names = {os.path.basename(p) for p in bench.KERNEL_SOURCES}
    kernel = re.compile(r"__global__[^;{]*\bcasclb_(step\w*|multistep)\s*\(")
    found = set()
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        text = open(path).read()
        if kernel.search(text):
            found.add(os.path.basename(path))
            found.update(h for h in re.findall(r'#include "(\w+\.hpp)"', text) if h != "kernels.hpp")   # declarations only
    assert {"kernels.hip", "step_flat.hip", "multistep.hip", "node.hpp", "lattice.hpp"} <= found
    assert found <= names, found - names


def test_steps_that_share_a_pass_have_no_share_of_the_memory_peak():
    assert bench.pct_hbm_peak("casclb_multistep<D2Q9_D2Q5,f32dev>", 10377.0) is None
    assert bench.pct_hbm_peak("casclb_step<D2Q9_D2Q5,f32dev>", 4000.0) == 50.0
