"""Detectors of their own in several threads, each on a stream of its own:
what the launches of one process share (kernels set up for their LDS, the
error text) serves them all.  Lists against the oracle."""
import threading

import numpy as np
import pytest
import torch

import paper_1803_11036_amd as ssd
import oracle
import tracegen as tg
from _parity import log
from test_gpu_close_tail import _pairs

pytestmark = pytest.mark.gpu


def test_detectors_in_threads():
    geo = [(12, 6, 5, 32), (12, 4, 6, 24), (10, 5, 5, 24), (9, 8, 3, 24)]
    slots = 4
    got, failed, start = {}, [], threading.Barrier(len(geo))

    def work(i):
        try:
            q, r, d, kb = geo[i]
            stream = torch.cuda.Stream(device="cuda:0")
            with torch.cuda.stream(stream):
                p = ssd.make_params(q=q, r=r, delta=d, eta=1024, k=2, theta=16, key_bits=kb, verify_rehash=True)
                det = ssd.init_detector(p, tg.hash_tables(i), device="cuda:0")
                ssd.set_tuning(det, ssd.SSD_TUNE_SCAN_MODE, ssd.SSD_SCAN_BINNED)
                ssd.set_tuning(det, ssd.SSD_TUNE_COUNTED_MIN_ITEMS, i)
                start.wait(60)
                for t in range(slots):
                    pairs = torch.from_numpy(_pairs(i, 20, 40, kb, t).view(np.int32)).to("cuda:0")
                    ssd.scan_slice(det, pairs, t)
                    got[i, t] = ssd.close_slice(det)
                stream.synchronize()
                det.destroy()
        except BaseException as e:      # noqa: BLE001 (shown by the test)
            failed.append((i, e))
            start.abort()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(geo))]
    for x in threads:
        x.start()
    for x in threads:
        x.join(60)
    assert not failed, failed
    for i, (q, r, d, kb) in enumerate(geo):
        o = oracle.RSEA(q, r, d, 1024, 2, 16, tg.hash_tables(i), key_bits=kb, verify_rehash=True)
        for t in range(slots):
            log(f"threads: detector {i} slot {t}")
            o.scan(_pairs(i, 20, 40, kb, t))
            ip, rk, _ = o.close()
            assert len(ip) >= 20
            assert np.array_equal(got[i, t]["ip"], ip) and np.array_equal(got[i, t]["rk"], rk)
