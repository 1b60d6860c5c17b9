"""The pass scan of a small state around the size from which it looks at a
sample of the call's hosts, and on both sides of what the sample decides:
distinct hosts, one, ten and a share of one around the quarter and the half of
the call, pairs that end before the sample's last stride and behind it.  Cells
equal to the oracle's."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,r,delta,cell_bits", [(12, 6, 5, 8), (10, 5, 8, 8), (10, 8, 4, 8), (11, 5, 6, 16),
                                                 (12, 4, 7, 8)])
def test_sampled_calls(q, r, delta, cell_bits):
    g, o = make_pair(q, r, delta, 1024, 3, 8192, tg.hash_tables(q * r), key_bits=24, rehash=True,
                     cell_bits=cell_bits)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_PASSES)
    rng = np.random.default_rng(q + r)
    for t, (n, share, hosts) in enumerate([((1 << 19) - 1, 0.0, 0), (1 << 19, 0.0, 0), ((1 << 19) + 63, 0.25, 1),
                                           (524_353, 0.5, 1), (600_001, 1.0, 10), (1 << 19, 1.0, 1)]):
        log(f"sampled call q={q} r={r} n={n} share={share}")
        p = rng.integers(0, 1 << 32, (n, 2), dtype=np.uint32)
        if share:
            few = rng.random(n) < share
            p[few, 0] = rng.integers(0, 1 << 32, hosts, dtype=np.uint32)[np.arange(int(few.sum())) % hosts]
        scan_both(g, o, p, t)
        compare_state(g, o)
        ssd.close_slice(g, advance_only=True)
        o.close(advance_only=True)
    g.destroy()
