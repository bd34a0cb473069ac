"""The bytes that bench.py charges a tet for are those of the library's element record."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_record_bytes():
    with open(os.path.join(ROOT, "paper_2104_02646_amd", "csrc", "gsim_internal.h")) as f:
        values = int(re.search(r"constexpr int REC_TET = (\d+);", f.read()).group(1))
    assert bench.RECORD_TET == 4 * values + 8  # and mu, lambda
    ne, np_, ntp, T, K = 1000, 300, 700, 20, 5
    timing = {k: (10, 1.0) for k in ("element_fwd", "element_adj", "element_dual")}
    table = bench.kernel_table(timing, ne, np_, ntp, T, K)
    fwd, adj, dual = (table[k]["compulsory_bytes_per_launch"] for k in timing)
    assert fwd == bench.RECORD_TET * ne + 36 * ntp
    assert adj == (bench.RECORD_TET + 16) * ne + 52 * ntp + 17 * ntp / T
    assert dual == fwd + adj - bench.RECORD_TET * ne  # a tile's two passes read its records once
    line = bench.roofline(table["element_dual"], "element_dual", None)
    assert line["achieved"] == dual / 1e-4 / 1e9 and line["frac"] == line["achieved"] / bench.HBM_PEAK_GBS
