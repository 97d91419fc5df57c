"""What bench.py ties its recorded profiles and rates to (no GPU)."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_1107_4543_amd", "csrc")


def test_the_source_hash_covers_every_step_kernel_and_what_it_includes():
    names = [n for n in sorted(os.listdir(CSRC)) if n.endswith((".hip", ".hpp"))]
    text = {n: open(os.path.join(CSRC, n)).read() for n in names}
    kernels = [n for n in names if re.search(r"__global__[^;{]*\bk_(step|pool|diag|project|init)", text[n])]
    assert "lbm_kernels.hip" in kernels and "lbm_tile.hip" in kernels
    for n in kernels:
        assert n in bench.KERNEL_SOURCES, n
        for h in re.findall(r'#include "(\w+\.hpp)"', text[n]):
            assert h in bench.KERNEL_SOURCES or h == "lbm_internal.hpp", (n, h)
