"""The benchmark's operation and byte counts of a Wilson-loop measurement against the counters of the
kernel that does it."""
import os
import re

import bench


def test_wilson_work_matches_the_counters():
    with open(os.path.join(bench.ROOT, "profiles", "wilson_kernel_48x48x48x48_counters.md")) as f:
        text = f.read()
    m = re.search(r"VALU (\d+), SALU \d+, VMEM reads ([0-9.]+)", text)
    valu, reads = int(m.group(1)), float(m.group(2))
    flop, gathered = bench.wilson_work(4)
    assert abs(gathered / 16 - reads) <= 0.01 * reads
    # one FMA an instruction, and at most half as many again for addresses and sums
    assert 0.65 * valu < flop / 2 <= valu
    assert f"gathers {gathered // 16} links" in text.replace("\n", " ")


def test_wilson_work_of_one_plaquette():
    """R = T = 1: A C and B D, one dot product, four links; six planes."""
    assert bench.wilson_work(1) == (6 * (2 * 16 + 4) * 2, 6 * 4 * 16)
