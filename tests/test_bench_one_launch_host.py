"""Roofline record of a workload whose compression steps all run in one launch:
no contraction class has any launch or time."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_roofline_without_contraction_launches():
    n = len(bench.CLASSES)
    launches, ms, flops, byts = [0] * n, [0.0] * n, [0.0] * n, [0.0] * n
    for cls, k, t, f, b in (("other", 11, 3.0, 3e9, 1e6), ("measure", 10, 0.1, 1e6, 1e5)):
        i = bench.CLASSES.index(cls)
        launches[i], ms[i], flops[i], byts[i] = k, t, f, b
    rl = bench.roofline((launches, ms, flops, byts), "c128")
    assert rl["kernel"] == "chain_kernel" and rl["launches"] == 11
    assert rl["unit"] == "TFLOP/s" and abs(rl["achieved"] - 1.0) < 1e-3
    assert rl["all_contraction_gemms"] is None
    # a few contraction launches beside other work: as before
    launches[0], ms[0], flops[0] = 2, 0.5, 1e9
    rl = bench.roofline((launches, ms, flops, byts), "c128")
    assert rl["unit"] == "GB/s" and rl["kernel"] == "other"
    assert abs(rl["all_contraction_gemms"]["achieved_tflops"] - 2.0) < 1e-3
