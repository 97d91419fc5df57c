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


def test_full_rate_is_one_fp32_operation_in_two_cycles_and_one_fp64_in_four():
    simds = 256 * 4
    assert bench.FULL_RATE["f32"] == simds * 64 / 2 * 2.4e9
    assert bench.FULL_RATE["f64"] == simds * 64 / 4 * 2.4e9
    r = bench.full_rate("f32", 23.9e12)
    assert abs(r["peak"] - 78.64) < 0.01 and abs(r["frac"] - 23.9 / 78.643) < 1e-4
    multi = bench.pool_roofline(7, 1 << 20, 10, 2.0)
    assert abs(multi["full_rate"]["frac"] - multi["frac"] / 2) < 1e-4
