"""Hot detection that reads a whole state, with plain and with streamed loads
(large states that the slice wrote much of): a quiet slice, a busy one, a
router merge.  R_k, hot lists and lists against the oracle."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,eta,cell_bits", [(14, 8192, 16), (14, 8192, 8)])
def test_quiet_and_busy_slices(q, eta, cell_bits):
    """768 MiB of 16-bit cells, streamed from 786432 named cells on; 384 MiB of 8-bit ones, from 98304 on."""
    g, o = make_pair(q, 3, 8, eta, 2, 200, tg.hash_tables(q), key_bits=22, rehash=True, cell_bits=cell_bits)
    if cell_bits == 8:
        ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED, 0)
    rng = np.random.default_rng(cell_bits)
    hosts = rng.integers(0, 1 << 22, 40_000, dtype=np.uint32)
    edge = (786_432 if cell_bits == 16 else 98_304) // 3
    for t, n in enumerate([3_000, edge - 1, edge, 3_000]):
        log(f"detection of {cell_bits}-bit cells, slice of {n} pairs")
        p = np.empty((n, 2), dtype=np.uint32)
        p[:, 0] = rng.choice(hosts, n)
        p[:2_000, 0] = hosts[:5][np.arange(2_000) % 5]
        p[:, 1] = rng.integers(0, 1 << 32, n, dtype=np.uint32)
        scan_both(g, o, p, t)
        assert len(close_both(g, o)) >= 5
        assert ssd.get_info(g)["counted"] == 0
    g.destroy()
