"""Closes are replayed as a HIP graph unless the caller turns it off: the first
close and the later ones, waited for and pipelined, and again after the knob
was off.  Lists against the oracle, launches by the phase timing."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import log, make_pair, scan_both
from test_gpu_close_tail import _pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pipelined", [False, True])
def test_closes_replay_the_graph(pipelined):
    g, o = make_pair(12, 6, 5, 1024, 3, 24, tg.hash_tables(5), rehash=True)
    ssd.set_tuning(g, ssd.SSD_TUNE_TIMING, 1)
    for t in range(6):
        log(f"close graph pipelined={pipelined} slot {t}")
        if t in (2, 4):
            ssd.set_tuning(g, ssd.SSD_TUNE_GRAPH, t == 4)
        scan_both(g, o, _pairs(t, 30, 40, 32, t), t)
        if pipelined:
            ssd.close_begin(g)
            got = ssd.close_end(g)
        else:
            got = ssd.close_slice(g)
        o.reconstruct()
        ip, rk, _ = o.results()
        assert np.array_equal(got["ip"], ip) and np.array_equal(got["rk"], rk), f"slot {t}"
        o.age()
        n = {k: v[1] for k, v in ssd.read_timing(g, reset=True).items()}
        off = t in (2, 3)
        assert n["close_graph"] == (0 if off else 1), f"slot {t}: {n}"
        assert [n[k] for k in ("hot_lists", "expand", "verify", "report")] == [1 if off else 0] * 4, f"slot {t}: {n}"
    g.destroy()
