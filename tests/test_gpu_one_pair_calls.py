"""Counted calls of one to three pairs: a binning segment of three to fifteen
offsets, whose staging is one pair of packed words.  State, R_k, hot lists and
lists against the oracle."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("q,r,delta,kb", [(12, 3, 6, 18), (12, 4, 6, 24), (12, 5, 6, 30)])
def test_counted_calls_of_a_pair(q, r, delta, kb, noalloc):
    log(f"one-pair calls r={r} noalloc={noalloc}")
    g, o = make_pair(q, r, delta, 1024, 2, 1, tg.hash_tables(r), key_bits=kb, rehash=True)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED_MIN_ITEMS, 0)
    scan = ssd.scan_slice_noalloc if noalloc else ssd.scan_slice
    rng = np.random.default_rng(r)
    reported = 0
    for t, sizes in enumerate([(1,), (1, 2), (3, 1, 1), (1,)]):
        for n in sizes:
            p = np.empty((n, 2), dtype=np.uint32)
            p[:, 0] = rng.integers(0, 1 << kb, n)
            p[:, 1] = rng.integers(0, 1 << 32, n, dtype=np.uint32)
            o.scan(p)
            scan(g, to_dev(p), t)
        compare_state(g, o)
        reported += len(close_both(g, o))
        assert ssd.get_info(g)["counted"] == 1, f"slice {t}"
    assert reported >= 8
    g.destroy()
