"""The expansion of several links in one launch: workgroups whose run of a
link's pairs is short look its hot bits up in memory, the others fill their
LDS with them, and links of both kinds, of every delta and of up to eight rows
meet in a launch.  Tuple counts, hot lists, R_k and lists against the
oracle."""
import numpy as np
import pytest

import oracle
import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import log, to_dev
from test_gpu_close_tail import _pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spec", [
    # q, r, delta, key_bits, hosts.  Short runs throughout, deltas 1 to 6, rows of half a word and of one.
    [(12, 6, 5, 32, 40), (14, 5, 6, 32, 30), (5, 6, 1, 9, 3), (10, 6, 2, 18, 8), (9, 5, 3, 18, 9), (5, 3, 3, 8, 4)],
    # 1025 hosts (about a million pairs of rows 0 and 1: full tables) between short runs
    [(12, 6, 5, 32, 20), (16, 6, 4, 32, 1025), (14, 5, 6, 32, 65), (8, 4, 4, 16, 25)],
    # up to eight rows: four waves a workgroup (keys of 24 bits: the hosts lie below 2^24)
    [(9, 8, 3, 24, 20), (10, 7, 3, 24, 40), (12, 6, 5, 32, 150), (9, 8, 1, 15, 12)]])
def test_links_of_a_launch(spec):
    spec = [(q, r, d, max(8, min(kb, (r - 2) * d + q)), h) for q, r, d, kb, h in spec]
    tabs = [tg.hash_tables(60 + i) for i in range(len(spec))]
    b = ssd.batch_init([ssd.make_params(q=q, r=r, delta=d, eta=1024, k=2, theta=16, key_bits=kb, verify_rehash=True,
                                        max_tuples=1 << 22) for q, r, d, kb, _ in spec], tabs, device="cuda:0")
    orcs = [oracle.RSEA(q, r, d, 1024, 2, 16, t, key_bits=kb, verify_rehash=True)
            for (q, r, d, kb, _), t in zip(spec, tabs)]
    total = 0
    for t in range(2):
        per = [_pairs(100 + i, h, 24, kb, t) for i, (q, r, d, kb, h) in enumerate(spec)]
        offs = np.zeros(len(per) + 1, dtype=np.uint64)
        offs[1:] = np.cumsum([len(p) for p in per])
        ssd.batch_scan(b, to_dev(np.concatenate(per)), offs, t)
        lists, status = ssd.batch_close(b)
        for i, o in enumerate(orcs):
            log(f"expansion of a batch, slice {t} link {i}: {len(lists[i])} hosts")
            o.scan(per[i])
            o.reconstruct()
            ip, rk, _ = o.results()
            assert status[i] == 0
            assert np.array_equal(lists[i]["ip"], ip) and np.array_equal(lists[i]["rk"], rk), f"slice {t} link {i}"
            assert np.array_equal(ssd.batch_read_rk(b, i), o.rk()), f"slice {t} link {i}"
            levels = ssd.batch_get_info(b, i)["level_counts"]
            assert levels[spec[i][1] - 3] == len(o.tuples()), f"slice {t} link {i}"
            total += len(ip)
            o.age()
    assert total > 50
    b.destroy()
