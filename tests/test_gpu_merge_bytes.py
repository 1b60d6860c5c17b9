"""The router merge on arbitrary state bytes: clocks before, at and after the
stamp wrap, windows of one slot to the largest (longer than the clock, so that
live stamps lie on both sides of the wrap), stale cells of every age, one to
more than 64 sources.  The merged bytes against the rule written out per cell:
the stamp of the smallest distance below k, else empty."""
import numpy as np
import pytest
import torch

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,cell_bits", [(1, 8), (8, 8), (100, 8), (254, 8), (300, 16)])
@pytest.mark.parametrize("n_routers", [1, 2, 16, 70])
def test_merge_bytes(k, cell_bits, n_routers):
    m, dt = (255, np.uint8) if cell_bits == 8 else (65535, np.uint16)
    p = ssd.make_params(q=5, r=3, delta=3, eta=1024, k=k, theta=10, key_bits=8, max_tuples=64, max_results=64,
                        cell_bits=cell_bits)
    tabs = tg.hash_tables(2)
    dets = [ssd.init_detector(p, tabs, device="cuda:0") for _ in range(n_routers + 1)]
    blob = ssd.export_state(dets[0])
    n = (blob.size - ssd.STATE_HEADER_BYTES) * 8 // cell_bits
    rng = np.random.default_rng(k + n_routers)
    for t in (0, 5, k - 1, k, m - 2, m - 1, m, m + 40):
        log(f"merge bytes k={k} routers={n_routers} slice {t}")
        cur = 1 + t % m
        best = np.full(n, m, dtype=np.int64)
        code = np.zeros(n, dtype=np.int64)
        for d in dets:
            # half the cells empty, the others of any stamp, many near the open slot's
            c = rng.integers(0, m + 1, n)
            near = (cur - 1 - rng.integers(0, min(k + 3, m), n)) % m + 1
            c = np.where(rng.random(n) < 0.5, 0, np.where(rng.random(n) < 0.5, c, near))
            b = blob.copy()
            b[64:72] = np.frombuffer(np.uint64(t).tobytes(), dtype=np.uint8)       # the open slice
            b[ssd.STATE_HEADER_BYTES:] = np.frombuffer(c.astype(dt).tobytes(), dtype=np.uint8)
            ssd.import_state(d, b)
            if d is not dets[0]:
                age = np.where(c == 0, m, (cur - c) % m)
                code = np.where(age < best, c, code)
                best = np.minimum(best, age)
        ssd.merge_router_state(dets[0], dets[1:])
        torch.cuda.synchronize()
        got = np.frombuffer(dets[0].state.cpu().numpy().tobytes(), dtype=dt)
        assert np.array_equal(got, np.where(best < k, code, 0)), f"slice {t}"
    for d in dets:
        d.destroy()
