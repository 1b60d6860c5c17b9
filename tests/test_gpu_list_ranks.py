"""Lists ranked by counting around the 32 keys of a ranking workgroup and the
128 keys that its reads are padded to, at the default limit; and the default
limit restored after another one."""
import numpy as np
import pytest

import paper_1803_11036_amd as ssd
import tracegen as tg
from _parity import close_both, log, make_pair, scan_both
from test_gpu_close_tail import _pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hosts", [31, 32, 33, 127, 128, 129])
def test_lists_around_a_workgroup(hosts):
    log(f"ranks of {hosts} hosts")
    g, o = make_pair(16, 6, 4, 1024, 1, 16, tg.hash_tables(11), rehash=True)
    scan_both(g, o, _pairs(hosts, hosts, 40, 32), 0)
    assert len(close_both(g, o)) == hosts
    g.destroy()


@pytest.mark.parametrize("graph", [0, 1])
def test_limit_restored(graph):
    """A list of about 9000 hosts, above the largest limit that can be set: after that limit it is ranked as if none
    had been set, in the same number of launches (a list above the limit takes one more, the multi-kernel sort)."""
    rng = np.random.default_rng(53000)
    p = np.empty((53000, 2), dtype=np.uint32)
    p[:, 0] = rng.integers(0, 1 << 15, 53000)
    p[:, 1] = rng.integers(0, 1 << 32, 53000, dtype=np.uint32)
    launches = {}
    for limits in ((), (64,), (64, 8192)):
        log(f"limits {limits}")
        g, o = make_pair(7, 4, 4, 1024, 1, 18, tg.hash_tables(11), key_bits=15, rehash=True, max_tuples=1 << 23)
        ssd.set_tuning(g, ssd.SSD_TUNE_GRAPH, graph)
        ssd.set_tuning(g, ssd.SSD_TUNE_TIMING, 1)
        for x in limits:
            ssd.set_tuning(g, ssd.SSD_TUNE_SORT_BLOCK_LIMIT, x)
        scan_both(g, o, p, 0)
        assert len(close_both(g, o, check_internals=False)) > 8192
        launches[limits] = {k: v[1] for k, v in ssd.read_timing(g).items()}
        with pytest.raises(ssd.SSDError) as e:
            ssd.set_tuning(g, ssd.SSD_TUNE_SORT_BLOCK_LIMIT, 8193)
        assert e.value.status == -1
        g.destroy()
    assert launches[(64, 8192)] == launches[()]
    assert launches[(64,)] != launches[()]
