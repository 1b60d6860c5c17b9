"""Uncounted binned stores where a workgroup's segments go from two to more:
calls of 84 segments over 1536 bins (two each), 85 and 86, and of more; and
five rows in bins of 2 MiB, which stay at two.  Cells equal to the oracle's."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,r,delta,bin_bytes", [(16, 6, 4, 1 << 18), (14, 5, 6, 1 << 21)])
def test_segments_of_a_workgroup(q, r, delta, bin_bytes):
    g, o = make_pair(q, r, delta, 1024, 2, 8192, tg.hash_tables(r), rehash=True)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED, 0)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_BIN_BYTES, bin_bytes)
    rng = np.random.default_rng(q)
    for t, sizes in enumerate([(84 * 2048, 84 * 2048 + 1), (86 * 2048 - 7, 600_001)]):
        for n in sizes:
            log(f"segments of a workgroup r={r} n={n}")
            p = rng.integers(0, 1 << 32, (n, 2), dtype=np.uint32)
            p[: n // 4, 0] = 77
            scan_both(g, o, p, t)
        compare_state(g, o)
        ssd.close_slice(g, advance_only=True)
        o.close(advance_only=True)
    g.destroy()
