"""The binning's two segment sizes (half a compute unit's LDS, a whole one's)
at their edges: register and general binning, calls of one pair, one short of
and one over a segment and a round of workgroups, bins whose runs are just too
short for half segments, bins of few estimators, 8- and
16-bit cells.  Cells and lists are equal to the oracle's."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,r,delta,eta,cell_bits,bin_bytes", [
    (14, 6, 5, 1024, 8, 1 << 18), (16, 6, 4, 1024, 8, 1 << 18), (14, 5, 6, 1024, 8, 1 << 20),
    (16, 5, 6, 1024, 8, 1 << 18), (14, 4, 9, 1024, 8, 1 << 19), (14, 9, 3, 1024, 8, 1 << 18),
    (10, 5, 8, 16384, 8, 1 << 18), (8, 6, 6, 1 << 16, 8, 1 << 18), (15, 5, 6, 1024, 16, 1 << 19)])
def test_segments_against_oracle(q, r, delta, eta, cell_bits, bin_bytes):
    g, o = make_pair(q, r, delta, eta, 3, 60, tg.hash_tables(q + r), rehash=True, cell_bits=cell_bits,
                     max_tuples=1 << 22)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED, 0)      # (small calls would keep counters in place of binning)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_BIN_BYTES, bin_bytes)
    rng = np.random.default_rng(q * r)
    hosts, heavy = rng.integers(0, 1 << 32, 3000, dtype=np.uint32), rng.integers(0, 1 << 32, 6, dtype=np.uint32)
    bins = (r << q) * eta * cell_bits // 8 // bin_bytes
    half = min((20480 - 32 - 2048 - bins - 1) // r, {6: 3072, 5: 4096}.get(r, 1 << 20))
    for t, sizes in enumerate([(1, half - 1, half), (half + 1, 2 * half + 1), (6145, 2049), (256 * 2048 + 1,)]):
        log(f"segments q={q} r={r} eta={eta} slice {t}: {sizes}")
        for n in sizes:
            p = np.empty((n, 2), dtype=np.uint32)
            p[:, 0] = rng.choice(hosts, n)
            p[:, 1] = rng.integers(0, 40, n)
            p[: n // 8, 0] = rng.choice(heavy, n // 8)
            p[: n // 8, 1] = rng.integers(0, 1 << 32, n // 8, dtype=np.uint32)
            scan_both(g, o, p, t)
        compare_state(g, o)
        if q >= 14:
            close_both(g, o)
        else:                        # (few columns: most are hot)
            ssd.close_slice(g, advance_only=True)
            o.close(advance_only=True)
    g.destroy()


@pytest.mark.parametrize("q,r,delta,full", [(16, 6, 4, 6144), (16, 5, 6, 7168), (16, 9, 3, 4063)])
def test_several_segments_a_workgroup(q, r, delta, full):
    """Calls of more whole segments than compute units, the last one ragged: workgroups take two or three in turn."""
    g, o = make_pair(q, r, delta, 1024, 2, 60, tg.hash_tables(r), rehash=True, max_tuples=1 << 22)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED, 0)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_BIN_BYTES, 1 << 18)
    rng = np.random.default_rng(r)
    hosts = rng.integers(0, 1 << 32, 1 << 16, dtype=np.uint32)
    for t, n in enumerate([256 * full + 1, 512 * full + 1023]):
        log(f"rounds q={q} r={r} n={n}")
        p = np.empty((n, 2), dtype=np.uint32)
        p[:, 0] = rng.choice(hosts, n)
        p[:, 1] = rng.integers(0, 1 << 32, n, dtype=np.uint32)
        scan_both(g, o, p, t)
        compare_state(g, o)
        ssd.close_slice(g, advance_only=True)
        o.close(advance_only=True)
    g.destroy()


@pytest.mark.parametrize("cell_bits", [8, 16])
def test_runs_shared_by_lanes(cell_bits):
    """The bitmap stores with 1, 2, 3, 511, 512 and 513 runs a bin: shared by 1024 lanes down to one, empty runs and
    runs of thousands of offsets, counters exact."""
    g, o = make_pair(14, 6, 5, 1024, 3, 60, tg.hash_tables(3), rehash=True, cell_bits=cell_bits, max_tuples=1 << 22)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_COUNTED_MIN_ITEMS, 1)
    rng = np.random.default_rng(1)
    hosts, heavy = rng.integers(0, 1 << 32, 3000, dtype=np.uint32), rng.integers(0, 1 << 32, 6, dtype=np.uint32)
    for t, runs in enumerate([1, 2, 3, 511, 512, 513]):
        n = 2048 * runs - 5
        log(f"shared runs bits={cell_bits} runs={runs}")
        p = np.empty((n, 2), dtype=np.uint32)
        p[:, 0] = rng.choice(hosts, n)
        p[:, 1] = rng.integers(0, 40, n)
        p[: n // 8, 0] = rng.choice(heavy, n // 8)
        p[: n // 8, 1] = rng.integers(0, 4000, n // 8)
        scan_both(g, o, p, t)
        compare_state(g, o)
        close_both(g, o)
    g.destroy()


@pytest.mark.parametrize("n", [700_001, 1_000_003, 1_600_007])
def test_calls_around_the_staging(n):
    """Calls that half segments take in one step, in one more step than whole ones (which are then taken), and that
    either take in several."""
    g, o = make_pair(12, 6, 5, 1024, 2, 60, tg.hash_tables(7), rehash=True, max_tuples=1 << 22)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
    ssd.set_tuning(g, ssd.SSD_TUNE_SCAN_BIN_BYTES, 1 << 18)
    rng = np.random.default_rng(n)
    hosts = rng.integers(0, 1 << 32, 20_000, dtype=np.uint32)
    for t in range(2):
        p = np.empty((n, 2), dtype=np.uint32)
        p[:, 0] = rng.choice(hosts, n)
        p[:, 1] = rng.integers(0, 1 << 32, n, dtype=np.uint32)
        scan_both(g, o, p, t)
        compare_state(g, o)
        ssd.close_slice(g, advance_only=True)
        o.close(advance_only=True)
    g.destroy()
