"""The work that users of the sliding super point detector have it do, as cases to time.

A case is one slot of a running deployment: the slot's (cip, oip) pairs lie on the GPU, the window is already full, and
one pass scans the pairs and closes the slot.  Four kinds of deployment, each over the range of sizes that the
repository's workloads have:

- ``single``: one monitored link with a detector of its own (8- or 16-bit cells, one or several scan calls per slot, a
  synchronous or a pipelined close, the scan that allocates nothing);
- ``routers``: edge routers that scan their own pairs, merged every slot into a global detector, which closes;
- ``batch``: many links on one clock, scanned and closed together;
- ``group``: served streams of uneven sizes, scanned and closed by group calls.

Traces: hosts of Pareto(1.2) degree and planted super points; a slot carries ``distinct`` different pairs and repeats
them uniformly up to ``pairs``, in random order, as packets repeat their flows.  A pass returns the reported hosts and,
where a program could hold on to it, the detector's updated state.
"""
import math

import numpy as np
import torch

import paper_1803_11036_amd as ssd

# (q, r, delta) of the repository's workloads
GEOMETRIES = ((12, 6, 5), (13, 6, 5), (14, 5, 6), (15, 5, 6), (16, 6, 4))
THETAS = (512, 1024, 2048, 4096, 8192)


def single(name, q, r, delta, eta, k, theta, pairs, distinct, cell_bits=8, calls=1, pipelined=False, noalloc=False,
           rehash=False):
    c = {"kind": "single", "q": q, "r": r, "delta": delta, "eta": eta, "k": k, "theta": theta, "pairs": pairs,
         "distinct": distinct, "cell_bits": cell_bits, "calls": calls, "pipelined": pipelined, "noalloc": noalloc,
         "rehash": rehash}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest site: a slot of a few thousand packets, where launches and the close's latency are everything
        single("small_site", 12, 6, 5, 1024, 4, 64, 4_099, 3_001),
        # the repository's small trace: a million packets into a state that the Infinity Cache holds
        single("tiny_slot", 12, 6, 5, 1024, 4, 1024, 1_000_000, 272_000),
        # a 40 Gb/s core link, one call per slot, its close pipelined with the next slot's scan
        single("core_link", 16, 6, 4, 4096, 10, 1024, 6_000_000, 1_480_000, pipelined=True),
        # the same link fed by several odd-sized calls, each too small to keep counters, closed synchronously
        single("core_link_calls", 16, 6, 4, 4096, 10, 1024, 1_200_007, 700_001, calls=6),
        # a loop that may not allocate: a medium link scanned from static staging, packets hardly repeating
        single("noalloc_link", 15, 5, 6, 4096, 16, 2048, 999_983, 500_009, noalloc=True, rehash=True),
        # a fast link whose every packet is a new pair (a scan or a reflection attack seen from the edge)
        single("unique_pairs", 16, 6, 4, 4096, 8, 1024, 2_000_003, 2_000_003, rehash=True),
        # the paper's own parameters: one-second slots, a window of 300 of them, 16-bit cells
        single("paper_window", 14, 5, 6, 2048, 300, 1024, 6_000_000, 20_000, cell_bits=16),
        # sixteen edge routers of 1 to 4 million packets a slot, merged and closed centrally
        {"name": "routers_16", "kind": "routers", "routers": 16, "q": 14, "r": 5, "delta": 6, "eta": 4096, "k": 8,
         "theta": 2048, "pairs": 2_700_000, "distinct": 60_000},
        # a small multi-link batch, every link too small for the binned scan
        {"name": "batch_small", "kind": "batch", "links": 24, "scale": 0.02, "seed": 3},
        # the benchmark's batch: 64 links of 0.2 to 8 million packets a slot
        {"name": "batch_64", "kind": "batch", "links": 64, "scale": 1.0, "seed": 5},
        # a serving loop's turn: streams of uneven sizes scanned together, and all their slots closed
        {"name": "group_served", "kind": "group", "members": 12, "scale": 1.0, "seed": 7},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("single", "routers", "batch", "group"), (0.64, 0.12, 0.12, 0.12))[0]
    if kind == "routers":
        n, k, pairs = rng.randint(2, 16), rng.randint(4, 12), _log_uniform(rng, 50_000, 2_700_000)
        distinct = min(_log_uniform(rng, pairs // 64 + 1, pairs), (2048 << 14) // (4 * k * n))
        return {"kind": "routers", "routers": n, "q": 14, "r": 5, "delta": 6, "eta": 4096, "k": k, "theta": 2048,
                "pairs": pairs, "distinct": distinct}
    if kind == "batch":
        return {"kind": "batch", "links": rng.randint(3, 40), "scale": math.exp(rng.uniform(math.log(0.01), 0.0)),
                "seed": rng.randrange(1 << 20)}
    if kind == "group":
        return {"kind": "group", "members": rng.randint(2, 16), "scale": math.exp(rng.uniform(math.log(0.02), 0.0)),
                "seed": rng.randrange(1 << 20)}
    wide = rng.random() < 0.2
    q, r, delta = rng.choice(GEOMETRIES[2:4] if wide else GEOMETRIES)
    k = rng.randint(255, 300) if wide else rng.randint(1, 32)
    pairs = _log_uniform(rng, 1_000, 1_500_000 if wide else 6_000_000) | 1
    distinct = max(1, _log_uniform(rng, pairs / 64 + 1, pairs))
    theta = 1024 if wide else rng.choice((256, 512, 1024, 2048, 4096))
    eta = max(2048 if wide else 1024, theta)
    distinct = max(1, min(distinct, (theta << q) // (4 * k)))         # as loaded as the repository's traces, at most
    return single(None, q, r, delta, eta, k, theta, pairs, distinct, cell_bits=16 if wide else 8,
                  calls=rng.choice((1, 1, 1, 2, 5)), pipelined=rng.random() < 0.3,
                  noalloc=not wide and pairs < 1_000_000 and rng.random() < 0.2, rehash=rng.random() < 0.5)


# ---------------------------------------------------------------- inputs


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _tables(seed):
    return np.random.default_rng(seed).integers(0, 1 << 32, 2048, dtype=np.uint32)


def _slots(seed, n_slots, pairs, distinct, theta, streams=1):
    """For each of n_slots slots, the pairs of every stream: int32 (pairs, 2) tensors, each of ``distinct`` different
    pairs.  All are drawn from one host population (Pareto degrees, and planted hosts of 2 to 4 theta peers a
    window)."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    window = distinct * n_slots * streams
    planted = int(max(1, min(50, 0.2 * window / (3.0 * theta))))
    hosts = max(50, int(window / 5.1))
    u = torch.rand(hosts, generator=g, device=dev, dtype=torch.float64).clamp_min(1e-12)
    deg = torch.floor(u ** (-1.0 / 1.2)).clamp_max(max(20.0, min(0.05 * window, 100_000.0)))
    pdeg = theta * (2.0 + 2.0 * torch.rand(planted, generator=g, device=dev, dtype=torch.float64))
    cum = torch.cumsum(torch.cat([deg, pdeg.clamp_max(0.2 * window)]), 0)
    ids = torch.arange(hosts + planted, device=dev, dtype=torch.int64)
    ip = (ids * 2654435761 + seed * 40503) & 0xFFFFFFFF
    ip = ip ^ (ip >> 15)
    out = []
    for _ in range(n_slots):
        slot = []
        for _ in range(streams):
            at = torch.rand(distinct, generator=g, device=dev, dtype=torch.float64) * cum[-1]
            h = torch.searchsorted(cum, at).clamp_max(hosts + planted - 1)
            peer = torch.randint(0, 1 << 32, (distinct,), generator=g, device=dev, dtype=torch.int64)
            pool = torch.stack([ip[h], peer], 1)
            pool = torch.where(pool >= 1 << 31, pool - (1 << 32), pool).to(torch.int32)
            if distinct < pairs:
                pool = pool[torch.randint(0, distinct, (pairs,), generator=g, device=dev)]
            slot.append(pool.contiguous())
        out.append(slot)
    return out


def _link_list(case):
    """The links of a batch or group case: parameters and sizes of one slot."""
    rs = np.random.default_rng(case["seed"])
    links = []
    for _ in range(case.get("links") or case["members"]):
        q, r, delta = GEOMETRIES[int(rs.integers(5))]
        theta = THETAS[int(rs.integers(5))]
        k = int(rs.integers(4, 65))
        lo, hi = (65_536, 4_194_304) if case["kind"] == "group" else (200_000, 8_000_000)
        pairs = max(2000, int(math.exp(rs.uniform(math.log(lo), math.log(hi))) * case["scale"]))
        repeat = 1.0 if case["kind"] == "group" else 2.0
        distinct = int(max(200, min(0.25 * (1 << q) * theta / k, pairs / repeat)))
        links.append({"q": q, "r": r, "delta": delta, "eta": max(1024, theta), "k": k, "theta": theta,
                      "pairs": pairs, "distinct": distinct})
    return links


SHARED_SLOTS = 4      # different slots of a batch or group case, cycled


def _inputs(case, seed):
    """(links, hash tables, slots): slots[i][l] is link or stream l's pairs in slot i."""
    if case["kind"] == "single":
        # a full window of slots, so that cycling them keeps the window as it is
        return [case], [_tables(seed)], _slots(seed, case["k"], case["pairs"], case["distinct"], case["theta"])
    if case["kind"] == "routers":
        # every router sees other flows of the same hosts, and its own amount of packets
        links = [dict(case) for _ in range(case["routers"])]
        slots = _slots(seed, case["k"], int(1.5 * case["pairs"]), case["distinct"], case["theta"], case["routers"])
        share = np.random.default_rng(seed).uniform(0.4, 1.5, case["routers"])
        slots = [[p[:int(case["pairs"] * f)] for p, f in zip(s, share)] for s in slots]
        return links, [_tables(seed)] * len(links), slots
    links = _link_list(case)
    per = [_slots(seed * 1000 + l, SHARED_SLOTS, c["pairs"], c["distinct"], c["theta"]) for l, c in enumerate(links)]
    return links, [_tables(seed * 1000 + l) for l in range(len(links))], [
        [p[i][0] for p in per] for i in range(SHARED_SLOTS)]


def _params(c):
    return ssd.make_params(q=c["q"], r=c["r"], delta=c["delta"], eta=c["eta"], k=c["k"], theta=c["theta"],
                           verify_rehash=c.get("rehash", False), max_tuples=1 << 21, max_results=1 << 18,
                           cell_bits=c.get("cell_bits", 8))


def prepare(case, seed):
    links, tables, slots = _inputs(case, seed)
    s = {"case": case, "t": 0, "pending": False, "report": np.zeros(ROOM, dtype=ssd.RESULT_DTYPE), "filled": 0}
    if case["kind"] == "single":
        s["det"] = ssd.init_detector(_params(case), tables[0])
        s["slots"] = [torch.tensor_split(p[0], case["calls"]) for p in slots]
    elif case["kind"] == "routers":
        s["routers"] = [ssd.init_detector(_params(c), t) for c, t in zip(links, tables)]
        s["det"] = ssd.init_detector(_params(case), tables[0])
        s["slots"] = slots
    else:
        s["slots"] = []
        for p in slots:
            offsets = np.zeros(len(p) + 1, dtype=np.uint64)
            offsets[1:] = np.cumsum([x.shape[0] for x in p])
            s["slots"].append((torch.cat(p).contiguous(), offsets))
        del slots
        if case["kind"] == "batch":
            s["batch"] = ssd.batch_init([_params(c) for c in links], tables)
        else:
            s["members"] = [ssd.init_detector(_params(c), t) for c, t in zip(links, tables)]
            s["group"] = ssd.group_init(len(links))
    for _ in range(len(s["slots"]) + 1):       # the window fills (and a pipelined close is pending)
        run(s)
    return s


# ---------------------------------------------------------------- one pass


ROOM = 1 << 18        # a program's array for the hosts reported in a slot (max_results of a detector)


def _report(s, lists):
    """The lists, one after another, into the program's array (zero behind them); its columns and the lists' lengths."""
    out, n = s["report"], 0
    for x in lists:
        out[n:n + len(x)] = x
        n += len(x)
    if n < s["filled"]:
        out[n:s["filled"]] = 0
    s["filled"] = n
    return {"ip": out["ip"], "rk": out["rk"], "est": out["est"],
            "counts": np.array([len(x) for x in lists], dtype=np.int64)}


NOTHING = np.empty(0, dtype=ssd.RESULT_DTYPE)


def run(s):
    case, t = s["case"], s["t"]
    now = s["slots"][t % len(s["slots"])]
    s["t"] = t + 1
    if case["kind"] == "single":
        det = s["det"]
        scan = ssd.scan_slice_noalloc if case["noalloc"] else ssd.scan_slice
        for part in now:
            scan(det, part, t)
        if case["pipelined"]:
            # the list of the slot before, collected while this slot's scan runs
            res = ssd.close_end(det) if s["pending"] else NOTHING
            ssd.close_begin(det)
            s["pending"] = True
        else:
            res = ssd.close_slice(det)
        return dict(_report(s, [res]), state=det.state)
    if case["kind"] == "routers":
        for det, part in zip(s["routers"], now):
            ssd.scan_slice(det, part, t)
        ssd.merge_router_state(s["det"], s["routers"])
        res = ssd.close_slice(s["det"])
        for det in s["routers"]:
            ssd.close_slice(det, advance_only=True)
        return dict(_report(s, [res]), state=s["det"].state)
    pairs, offsets = now
    if case["kind"] == "batch":
        ssd.batch_scan(s["batch"], pairs, offsets, t)
        lists, status = ssd.batch_close_end(s["batch"]) if s["pending"] else ([NOTHING], [0])
        ssd.batch_close_begin(s["batch"])
    else:
        ssd.group_scan(s["group"], s["members"], pairs, offsets, [t] * len(s["members"]))
        lists, status = ssd.group_close_end(s["group"]) if s["pending"] else ([NOTHING], [0])
        ssd.group_close_begin(s["group"], s["members"])
    s["pending"] = True
    return dict(_report(s, lists), status=np.array(status, dtype=np.int64))


# ---------------------------------------------------------------- work and reference


def work(case):
    """The pairs read once, the touched cells written once, and for routers the states that are merged."""
    links = _link_list(case) if case["kind"] in ("batch", "group") else [case] * case.get("routers", 1)
    n = 0.0
    for c in links:
        n += 8.0 * c["pairs"] + c["r"] * c["distinct"] * (2.0 if c.get("cell_bits") == 16 else 1.0)
    if case["kind"] == "routers":
        n += (case["routers"] + 1.0) * (case["r"] << case["q"]) * case["eta"]
    return {"bytes": n, "flops": 0.0}


def _hash(table, x):
    return table[0][x & 255] ^ table[1][(x >> 8) & 255] ^ table[2][(x >> 16) & 255] ^ table[3][x >> 24]


def _reported(c, tables, window):
    """The hosts reported at the close of a window: the paper's method on whole sets, ascending by ip."""
    dev = _device()
    q, r, delta, eta, theta = c["q"], c["r"], c["delta"], c["eta"], c["theta"]
    qm, sh = (1 << q) - 1, q - delta
    km = (1 << sh) - 1
    need = math.ceil(eta * (1.0 - math.exp(-theta / eta)))
    tab = torch.from_numpy(tables.astype(np.int64)).to(dev).view(2, 4, 256)
    hot, cells = [], []
    for row in range(r):
        live = torch.zeros(eta << q, dtype=torch.bool, device=dev)
        for p in window:
            x = p.to(torch.int64) & 0xFFFFFFFF
            h0, d = _hash(tab[0], x[:, 0]) & qm, _hash(tab[1], x[:, 1]) & (eta - 1)
            col = h0 if row == 0 else ((x[:, 0] >> min(32, (row - 1) * delta)) ^ h0) & qm
            live[col * eta + d] = True
        live = live.view(1 << q, eta)
        hot.append(torch.nonzero(live.sum(1) >= need).flatten())
        cells.append(live[hot[-1]])
        del live
    he0 = hot[0].repeat_interleave(len(hot[1]))
    x = (he0 ^ hot[1].repeat(len(hot[0]))) & qm
    keep = x < 1 << 32
    he0, x = he0[keep], x[keep]
    for row in range(2, r):
        key, order = torch.sort(hot[row] & km)
        want = ((((x >> ((row - 2) * delta)) & qm) >> delta) ^ he0) & km
        lo, hi = torch.searchsorted(key, want), torch.searchsorted(key, want, right=True)
        n = hi - lo
        first = torch.repeat_interleave(torch.cumsum(n, 0) - n, n)
        at = torch.repeat_interleave(lo, n) + torch.arange(int(n.sum()), device=dev) - first
        he0, x = torch.repeat_interleave(he0, n), torch.repeat_interleave(x, n)
        top = ((he0 >> sh) ^ (hot[row][order[at]] >> sh)) & ((1 << delta) - 1)
        x = x | (top << ((row - 2) * delta + q))
        keep = x < 1 << 32
        he0, x = he0[keep], x[keep]
    if c.get("rehash", False):
        keep = (_hash(tab[0], x) & qm) == he0
        he0, x = he0[keep], x[keep]
    count = []
    for i in range(0, len(x), 4096):
        both = None
        for row in range(r):
            col = he0[i:i + 4096] if row == 0 else ((x[i:i + 4096] >> ((row - 1) * delta)) & qm) ^ he0[i:i + 4096]
            v = cells[row][torch.searchsorted(hot[row], col)]
            both = v if both is None else both & v
        count.append(both.sum(1))
    rk = torch.cat(count) if count else x[:0]
    x, rk = x[rk >= need].cpu().numpy(), rk[rk >= need].cpu().numpy()
    order = np.lexsort((-rk, x))
    x, rk = x[order], rk[order]
    first = np.concatenate([[True], x[1:] != x[:-1]]) if len(x) else np.zeros(0, dtype=bool)
    return x[first], rk[first]


def exact(case, seed):
    links, tables, slots = _inputs(case, seed)
    late = case["kind"] in ("batch", "group") or case.get("pipelined", False)
    t = len(slots) + 1 - (1 if late else 0)              # the slot whose list the first pass after prepare() returns
    window = range(max(0, t - case["k"] + 1) if "k" in case else 0, t + 1)
    ip, rk, est = [], [], []
    for l in range(1 if case["kind"] == "routers" else len(links)):
        c = links[l]
        used = sorted({i % len(slots) for i in window})
        parts = [p for i in used for p in (slots[i] if case["kind"] == "routers" else [slots[i][l]])]
        a, b = _reported(c, tables[l], parts)
        ip.append(a)
        rk.append(b)
        est.append(-float(c["eta"]) * np.log(np.maximum(c["eta"] - b.astype(np.float64), 1.0) / c["eta"]))
    out = np.zeros(ROOM, dtype=ssd.RESULT_DTYPE)
    n = sum(len(a) for a in ip)
    out["ip"][:n], out["rk"][:n], out["est"][:n] = np.concatenate(ip), np.concatenate(rk), np.concatenate(est)
    same = {"ip": out["ip"], "rk": out["rk"], "est": out["est"], "counts": np.array([len(a) for a in ip], np.int64)}
    return dict(same, status=None) if case["kind"] in ("batch", "group") else dict(same, state=None)
