"""The direct counted scan: small calls into large states that keep the
per-slot counters exact pair by pair -- of a single detector, and as counted
tiles of batches and groups -- at its edges: one pair and one wave, rows in
one and two groups of six, the same pairs many times over (one stamp
exchanged by many threads), cells of one 32-bit word, slices of several calls,
slices that outgrow it (the state is read instead) and windows of one slot.
State, R_k, hot lists and lists against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, compare_state, log, make_pair, scan_both, to_dev

pytestmark = pytest.mark.gpu


def _slice(rng, n, hosts, heavy):
    """n pairs of `hosts` light hosts and a few heavy ones, repeated about threefold."""
    d = np.empty((max(1, n // 3), 2), dtype=np.uint32)
    d[:, 0] = rng.choice(hosts, len(d))
    k = len(d) // 4
    d[:k, 0] = rng.choice(heavy, k)
    d[:, 1] = rng.integers(0, 1 << 32, len(d), dtype=np.uint32)
    return d[rng.integers(0, len(d), n)]


@pytest.mark.parametrize("q,r,delta,eta,k", [(16, 6, 4, 1024, 3), (16, 5, 6, 1024, 1), (15, 8, 3, 2048, 17),
                                             (15, 12, 2, 1024, 5)])
def test_single_detector(q, r, delta, eta, k):
    g, o = make_pair(q, r, delta, eta, k, 48, tg.hash_tables(5), rehash=True)
    rng = np.random.default_rng(q * r)
    hosts, heavy = rng.integers(0, 1 << 32, 4000, dtype=np.uint32), rng.integers(0, 1 << 32, 12, dtype=np.uint32)
    limit = ((r << q) * eta // 4096) // r                 # pairs a slice may bring
    # sizes of a slice's calls -> detection path (1 counters, 0 the state read)
    plan = [([1], 1), ([64, 65], 1), ([257, 3000, 1], 1), ([limit - 1], 1), ([5000], 1), ([limit + 1], 0), ([2000], 0)]
    for t, (sizes, path) in enumerate(plan):
        log(f"direct q={q} r={r} slice {t}: {sizes}")
        for n in sizes:
            scan_both(g, o, _slice(rng, n, hosts, heavy), t)
        compare_state(g, o)
        close_both(g, o)
        assert ssd.get_info(g)["counted"] == path, f"slice {t}"
    g.destroy()


def test_one_cell_many_threads():
    """Every pair the same, then pairs of one host whose cells share words: each cell counted once."""
    g, o = make_pair(16, 6, 4, 1024, 2, 16, tg.hash_tables(9))
    rng = np.random.default_rng(1)
    for t in range(3):
        p = np.full((16_000, 2), 77, dtype=np.uint32)       # within the slice's limit, 16384
        p[8_000:, 1] = rng.integers(0, 3000, 8_000)
        scan_both(g, o, p, t)
        compare_state(g, o)
        close_both(g, o)
        assert ssd.get_info(g)["counted"] == 1
    g.destroy()


def test_batch_and_group_tiles():
    """Links of a batch and members of a group in counted tiles beside uncounted
    ones and binned ones, the stamps wrapping (k + 1 slots of one window are
    enough for every counter move; 260 slots for the wrap)."""
    spec = [(15, 5, 6, 1024, 6, 7000), (14, 6, 5, 1024, 3, 9000), (12, 6, 5, 1024, 4, 9000), (14, 5, 6, 1024, 250, 8000),
            (15, 5, 6, 1024, 2, 70_000)]
    params = [ssd.make_params(q=q, r=r, delta=d, eta=e, k=k, theta=100, verify_rehash=True) for q, r, d, e, k, _ in spec]
    tabs = [tg.hash_tables(70 + i) for i in range(len(spec))]
    b = ssd.batch_init(params, tabs, device="cuda:0")
    members = [ssd.init_detector(p, t, device="cuda:0") for p, t in zip(params, tabs)]
    grp = ssd.group_init(len(spec), device="cuda:0")
    orcs = [oracle.RSEA(q, r, d, e, k, 100, tabs[i], verify_rehash=True) for i, (q, r, d, e, k, _) in enumerate(spec)]
    rng = np.random.default_rng(3)
    hosts = [rng.integers(0, 1 << 32, 3000, dtype=np.uint32) for _ in spec]
    heavy = [rng.integers(0, 1 << 32, 6, dtype=np.uint32) for _ in spec]
    total = 0
    for t in range(262):
        full = t < 8 or t > 252                           # between: one pair a link, so that the clock passes the wrap
        per = [_slice(rng, x[5] if full else 1, hosts[i], heavy[i]) for i, x in enumerate(spec)]
        offs = np.zeros(len(per) + 1, dtype=np.uint64)
        offs[1:] = np.cumsum([len(p) for p in per])
        dev = to_dev(np.concatenate(per))
        ssd.batch_scan(b, dev, offs, t)
        ssd.group_scan(grp, members, dev, offs, [t] * len(spec))
        lists, _ = ssd.batch_close(b)
        glists, _ = ssd.group_close(grp, members)
        for i, o in enumerate(orcs):
            o.scan(per[i])
            if full:
                o.reconstruct()
                ip, rk, _est = o.results()
                for name, got in (("batch", lists[i]), ("group", glists[i])):
                    assert np.array_equal(got["ip"], ip) and np.array_equal(got["rk"], rk), f"slice {t} {name} {i}"
                assert np.array_equal(ssd.batch_read_rk(b, i), o.rk()), f"slice {t} link {i}"
                assert np.array_equal(ssd.read_rk(members[i]), o.rk()), f"slice {t} member {i}"
                total += len(ip)
            o.age()
        if t < 8:
            got = [ssd.batch_get_info(b, i)["counted"] for i in range(len(spec))]
            assert got[0] == got[1] == 1 and got[2] == got[3] == 0, got
            assert [ssd.get_info(m)["counted"] for m in members[:4]] == got[:4]
    assert total > 50
    grp.destroy()
    b.destroy()
    for m in members:
        m.destroy()
