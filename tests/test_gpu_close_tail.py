"""The close's candidate expansion, final test and list ranking at the sizes
where their kernels change path: rows and deltas of the queue walk and of the
nested walk, waves with more full tuples than they stage, hot lists longer
than the LDS copy, estimators of one to many loads per lane, lists around a limit
set to 64 and with hosts regained several times.  Every product
against the oracle, bit for bit."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both

pytestmark = pytest.mark.gpu


def _pairs(seed, hosts, peers, key_bits, t=0):
    """Slot t's pairs: `peers` peers for each of `hosts` distinct hosts below 2^key_bits (the same in every slot)."""
    rng = np.random.default_rng(seed)
    ip = rng.choice(1 << min(key_bits, 24), hosts, replace=False).astype(np.uint64)
    if key_bits > 24:
        ip = (ip * 2654435761) % (1 << 32)
    rng = np.random.default_rng([seed, t])
    p = np.empty((hosts * peers, 2), dtype=np.uint32)
    p[:, 0] = np.repeat(ip, peers).astype(np.uint32)
    p[:, 1] = rng.integers(0, 1 << 32, hosts * peers, dtype=np.uint32)
    return p[rng.permutation(len(p))]


CASES = [
    # q, r, delta, key_bits, hosts, rehash
    (8, 4, 4, 16, 120, False),       # crowded rows: hundreds of thousands of full tuples
    (8, 4, 4, 16, 25, False),        # thousands of full tuples a workgroup, a few hundred keys
    (12, 6, 5, 32, 150, False),      # the small trace's geometry, hosts regained by false tuples
    (13, 6, 5, 32, 64, True),        # candidates with bits beyond the 32-bit key
    (14, 5, 6, 32, 65, False),       # 64-bit words of candidates
    (16, 6, 4, 32, 1025, True),      # the core link's geometry
    (10, 7, 3, 25, 40, False),       # seven rows: four waves a workgroup
    (9, 8, 3, 27, 20, False),        # eight rows
    (9, 8, 1, 15, 30, True),         # one overlap bit a row
    (12, 3, 6, 18, 200, False),      # three rows: no partial tuples
    (12, 4, 7, 26, 100, False),      # delta above 6: the nested walk
    (17, 3, 3, 20, 2100, True),      # hot lists longer than the LDS copy
    (18, 6, 3, 30, 100, False),      # hot bits larger than the LDS: the nested walk
    (5, 3, 3, 8, 6, False),          # rows of one word
    (4, 7, 1, 9, 5, True),           # rows of half a word
]


@pytest.mark.parametrize("q,r,delta,key_bits,hosts,rehash", CASES)
def test_expansion_against_oracle(q, r, delta, key_bits, hosts, rehash):
    log(f"expansion q={q} r={r} delta={delta} hosts={hosts}")
    g, o = make_pair(q, r, delta, 1024, 2, 16, tg.hash_tables(7), key_bits=key_bits, rehash=rehash,
                     max_tuples=1 << 22)
    for t in range(2):
        scan_both(g, o, _pairs(q * 100 + r, hosts, 24, key_bits, t), t)
        close_both(g, o)
    g.destroy()


@pytest.mark.parametrize("log2eta", [10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("r,delta,q", [(3, 8, 10), (6, 3, 8), (9, 2, 6)])
def test_final_test_against_oracle(log2eta, r, delta, q):
    """Lanes per tuple from 8 to 64, several loads a lane above 2^13; rows that fill one to three groups of three."""
    log(f"final test eta=2^{log2eta} r={r}")
    kb = (r - 2) * delta + q
    eta = 1 << log2eta
    g, o = make_pair(q, r, delta, eta, 1, 64, tg.hash_tables(3), key_bits=kb, max_tuples=1 << 20)
    scan_both(g, o, _pairs(log2eta, 12, 150, kb), 0)
    close_both(g, o)
    g.destroy()


@pytest.mark.parametrize("hosts", [0, 1, 63, 64, 65, 128, 1000])
@pytest.mark.parametrize("limit", [8192, 64])
def test_list_sizes(hosts, limit):
    """Short and long lists, also around a limit above which the multi-kernel sort takes them."""
    log(f"list of {hosts} hosts, limit {limit}")
    g, o = make_pair(16, 6, 4, 1024, 1, 16, tg.hash_tables(11), rehash=True)
    ssd.set_tuning(g, ssd.SSD_TUNE_SORT_BLOCK_LIMIT, limit)
    scan_both(g, o, _pairs(hosts, hosts, 24, 32), 0)
    res = close_both(g, o)
    assert len(res) >= hosts * 0.9
    g.destroy()


@pytest.mark.parametrize("q,r,delta,kb,theta,rehash,n", [
    (7, 4, 4, 15, 18, True, 52500), (7, 4, 4, 15, 18, True, 53000), (7, 4, 4, 15, 18, True, 55500),
    (7, 4, 4, 15, 18, True, 55700), (6, 5, 3, 14, 10, False, 24000)])
def test_long_lists(q, r, delta, kb, theta, rehash, n):
    """Crowded estimators that accept 8100, 9095, 15310 and 15640 hosts (lists ranked by counting hold 15360 keys), and
    about 9000 keys of 7000 hosts that false tuples regain."""
    log(f"long list q={q} n={n}")
    g, o = make_pair(q, r, delta, 1024, 1, theta, tg.hash_tables(11), key_bits=kb, rehash=rehash, max_tuples=1 << 23)
    rng = np.random.default_rng(n)
    p = np.empty((n, 2), dtype=np.uint32)
    p[:, 0] = rng.integers(0, 1 << kb, n)
    p[:, 1] = rng.integers(0, 1 << 32, n, dtype=np.uint32)
    scan_both(g, o, p, 0)
    close_both(g, o)
    g.destroy()


@pytest.mark.parametrize("q,r,delta", [(12, 6, 5), (8, 12, 2)])
def test_closes_of_both_kinds(q, r, delta):
    """Waited-for and pipelined closes in turn, replayed as a graph or (knob off) launched directly: lists as the
    oracle's."""
    kb = min(32, (r - 2) * delta + q)
    g, o = make_pair(q, r, delta, 1024, 3, 24, tg.hash_tables(5), key_bits=kb, rehash=True, max_tuples=1 << 22)
    for t in range(9):
        log(f"close kinds r={r} slot {t}")
        if t in (5, 7):
            ssd.set_tuning(g, ssd.SSD_TUNE_GRAPH, t == 7)
        scan_both(g, o, _pairs(t, 30, 40, kb, t), t)
        if t % 3 == 1:
            ssd.close_begin(g)
            got = ssd.close_end(g)
            o.reconstruct()
            ip, rk, _ = o.results()
            assert np.array_equal(got["ip"], ip) and np.array_equal(got["rk"], rk)
            o.age()
        else:
            close_both(g, o)
    g.destroy()


@pytest.mark.parametrize("cell_bits,k", [(8, 3), (8, 20), (16, 5)])
def test_slots_prepared_by_the_close_before(cell_bits, k):
    """A close leaves the next slot's constants and cleared bitmasks: past the wraps of the stamps and of the expiry
    phase, and after everything that moves the clock another way (advance-only slots, group closes, a resumed state)."""
    def fresh():
        return make_pair(8, 4, 4, 1024, k, 30, tg.hash_tables(2), key_bits=16, rehash=True, cell_bits=cell_bits,
                         max_tuples=1 << 20)
    g, o = fresh()
    group = ssd.Group(4) if cell_bits == 8 else None
    for t in range(530):
        kind = "own" if t % 7 else ("advance", "group", "begin", "resume")[t // 7 % 4]
        if kind == "group" and group is None:
            kind = "own"
        if kind == "resume":
            blob = ssd.export_state(g)
            g.destroy()
            g = fresh()[0]
            ssd.import_state(g, blob)
        if t % 3 == 0 or t % 7 < 2:
            scan_both(g, o, _pairs(t, 6, 60, 16, t), t)
        o.reconstruct()
        ip, rk, _ = o.results()
        if kind == "advance":
            ssd.close_slice(g, advance_only=True)
        else:
            if kind == "group":
                lists, status = ssd.group_close(group, [g])
                assert status[0] == 0
                got = lists[0]
            elif kind == "begin":
                ssd.close_begin(g)
                got = ssd.close_end(g)
            else:
                got = ssd.close_slice(g)
            assert np.array_equal(got["ip"], ip) and np.array_equal(got["rk"], rk), f"slot {t} ({kind})"
        o.age()
        if t % 50 == 49:
            log(f"prepared slots bits={cell_bits} k={k} slot {t}")
            compare_state(g, o)
    g.destroy()
