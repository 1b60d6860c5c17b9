"""The direct counted scan's counters where a wave's lanes move the same ones:
calls of one host, of as many as a wave adds for together and one more, of a
heavy host among light ones; cells whose old stamps have
different ages, and none.  State, R_k, hot lists and lists against the
oracle."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hosts,heavy", [(1, 0.0), (12, 0.0), (13, 0.0), (4000, 0.5)])
def test_counters_moved_together(hosts, heavy):
    g, o = make_pair(16, 6, 4, 1024, 4, 300, tg.hash_tables(4), rehash=True)
    rng = np.random.default_rng(hosts)
    ip = rng.integers(0, 1 << 32, hosts, dtype=np.uint32)
    for t in range(7):
        log(f"counters moved together, {hosts} hosts, {heavy} heavy, slice {t}")
        for n in (1, 63, 8_000) if t % 3 else (64, 2_000):
            p = np.empty((n, 2), dtype=np.uint32)
            p[:, 0] = ip[np.arange(n) % hosts]
            p[rng.random(n) < heavy, 0] = ip[0]
            p[:, 1] = rng.integers(0, 3000, n)      # (cells come back after one to three slices)
            scan_both(g, o, p, t)
        compare_state(g, o)
        close_both(g, o)
        assert ssd.get_info(g)["counted"] == 1
    g.destroy()
