"""The pass scan by eighths of a small state: sizes around its pair bound,
rows that split over two eighths and eighths of several rows, states up to its
size bound and one above, 8- and 16-bit cells, pass windows smaller than the
state: state and lists against the oracle."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,r,delta,eta,cell_bits,pass_bytes", [
    (12, 6, 5, 1024, 8, None), (12, 6, 5, 1024, 8, 5 << 20), (13, 3, 8, 1024, 8, None), (11, 12, 2, 1024, 8, None),
    (4, 3, 2, 1024, 8, None), (11, 5, 6, 1024, 16, None), (12, 7, 4, 1024, 8, None)])
def test_eighths_against_oracle(q, r, delta, eta, cell_bits, pass_bytes):
    kb = max(8, min(32, (r - 2) * delta + q)) if q > 4 else 8
    if (r - 2) * delta + q < kb:
        r = 4
    g, o = make_pair(q, r, delta, eta, 3, 200, tg.hash_tables(8), key_bits=kb, rehash=True, cell_bits=cell_bits,
                     max_tuples=1 << 22)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_PASSES)
    if pass_bytes:
        ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_PASS_BYTES, pass_bytes)
    rng = np.random.default_rng(q + r)
    hosts = rng.integers(0, 1 << kb, 300, dtype=np.uint64).astype(np.uint32)
    for t, n in enumerate([(1 << 16) - 1, 1 << 16, 200_001]):
        log(f"eighths q={q} r={r} n={n}")
        p = np.empty((n, 2), dtype=np.uint32)
        p[:, 0] = rng.choice(hosts, n)
        p[:, 1] = rng.integers(0, 60, n)
        p[: n // 8, 0] = hosts[:5][rng.integers(0, 5, n // 8)]
        p[: n // 8, 1] = rng.integers(0, 1 << 32, n // 8, dtype=np.uint32)
        scan_both(g, o, p, t)
        compare_state(g, o)
        if q > 4:                    # (16 columns are all hot)
            close_both(g, o)
        else:
            ssd.close_slice(g, advance_only=True)
            o.close(advance_only=True)
    g.destroy()
