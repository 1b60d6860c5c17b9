"""Slots that only advance: the dead cells of the slot's expiry phase cleared
and the clock moved, with 8- and 16-bit cells, the smallest and the largest
estimators, every estimator in the phase and one in many, past the stamps'
wrap, between scans and before a close.  Cells are equal to the oracle's."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,r,eta,k,cell_bits,slots", [
    (8, 3, 1024, 254, 8, 600), (9, 4, 4096, 250, 8, 530), (8, 3, 65536, 3, 8, 300), (10, 5, 2048, 100, 8, 300),
    (15, 4, 1024, 3, 16, 12), (8, 3, 65536, 2, 16, 12), (8, 3, 1024, 300, 16, 320)])
def test_advance_against_oracle(q, r, eta, k, cell_bits, slots):
    g, o = make_pair(q, r, 4, eta, k, 8, tg.hash_tables(q), key_bits=8, rehash=True, cell_bits=cell_bits,
                     max_tuples=1 << 22)
    rng = np.random.default_rng(k)
    for t in range(slots):
        if t % max(1, slots // 6) < 2:
            log(f"advance q={q} eta={eta} k={k} bits={cell_bits} slot {t}")
            p = rng.integers(0, 1 << 32, (60_000, 2), dtype=np.uint32)
            p[:, 0] &= 0xFF
            scan_both(g, o, p, t)
        ssd.close_slice(g, advance_only=True)
        o.close(advance_only=True)
        if t % max(1, slots // 6) < 8:
            compare_state(g, o)
            # the phase's estimators hold the window's stamps only
            top = 255 if cell_bits == 8 else 65535
            raw = g.state.cpu().numpy().view(np.uint8 if cell_bits == 8 else np.uint16).reshape(r << q, eta)[t % (top - k)::top - k]
            window = [0] + [1 + s % top for s in range(max(0, t - k + 1), t + 1)]
            assert np.isin(raw, np.array(window, dtype=raw.dtype)).all(), f"slot {t}: dead cells left in its phase"
    compare_state(g, o)
    close_both(g, o)
    compare_state(g, o)
    g.destroy()
