"""A batch's binned links side by side in one staging: binning segments whose
offsets are no multiple of four (five rows), in odd numbers, so that every link but the first would start off the 16 bytes that
segments are written and read in; and one link alone.  R_k and lists against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spec", [
    # q, r, delta, eta, pairs: 19, 22 and 21 segments of 3647 pairs of five rows
    [(14, 5, 6, 1024, 66_000), (14, 5, 6, 1024, 80_001), (14, 5, 6, 1024, 73_000), (12, 6, 5, 1024, 66_001)],
    # 19 segments of 3615, then links of six and nine rows
    [(15, 5, 6, 1024, 65_536), (16, 6, 4, 1024, 70_001), (14, 9, 3, 1024, 70_001)],
    # a batch of one link, which takes the same launches
    [(12, 6, 5, 1024, 66_001)]])
def test_links_side_by_side(spec):
    theta, k = 100, 2
    tabs = [tg.hash_tables(40 + i) for i in range(len(spec))]
    b = ssd.batch_init([ssd.make_params(q=q, r=r, delta=d, eta=e, k=k, theta=theta, verify_rehash=True)
                        for q, r, d, e, _ in spec], tabs, device="cuda:0")
    orcs = [oracle.RSEA(q, r, d, e, k, theta, t, verify_rehash=True) for (q, r, d, e, _), t in zip(spec, tabs)]
    rng = np.random.default_rng(len(spec))
    hosts, heavy = rng.integers(0, 1 << 32, 5000, dtype=np.uint32), rng.integers(0, 1 << 32, 8, dtype=np.uint32)
    total = 0
    for t in range(3):
        log(f"links side by side, slice {t}")
        per = []
        for x in spec:
            p = np.empty((x[4], 2), dtype=np.uint32)
            p[:, 0] = rng.choice(hosts, len(p))
            p[: len(p) // 8, 0] = rng.choice(heavy, len(p) // 8)
            p[:, 1] = rng.integers(0, 600, len(p))
            per.append(p[rng.permutation(len(p))])
        offs = np.zeros(len(per) + 1, dtype=np.uint64)
        offs[1:] = np.cumsum([len(p) for p in per])
        ssd.batch_scan(b, to_dev(np.concatenate(per)), offs, t)
        lists, status = ssd.batch_close(b)
        for i, o in enumerate(orcs):
            o.scan(per[i])
            o.reconstruct()
            ip, rk, _ = o.results()
            assert status[i] == 0
            assert np.array_equal(lists[i]["ip"], ip) and np.array_equal(lists[i]["rk"], rk), f"slice {t} link {i}"
            assert np.array_equal(ssd.batch_read_rk(b, i), o.rk()), f"slice {t} link {i}"
            total += len(ip)
            o.age()
    assert total >= 3 * len(spec)
    b.destroy()
