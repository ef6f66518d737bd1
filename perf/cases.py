"""The work a user of this library has it do, as cases to time.

Every case goes through the package's public calls: searches of [1, N], range queries at the
magnitudes of the served and batched workloads (starts below 2^40), batches of queries, a
burst of served requests, and plain radicals on the host and on the device.  Sizes are
those of bench.py, the tests and the input generators (queries of 2^10 .. 2^24 integers in
batches, requests of 2^12 .. 2^28 when served, N up to 2^36), with odd ones among them.
A case fixes the sizes; the seed sets where the ranges lie (or N's last digits).
"""
import math
import random

import numpy as np
import torch

from paper_2506_01099_amd import Benelux, Server

_kept = {}


def _context():
    """One context per process, as a program that makes many calls keeps it."""
    if "ctx" not in _kept:
        _kept["ctx"] = Benelux(device=0)
    return _kept["ctx"]


def _server():
    """Two lanes over a context of their own, started once."""
    if "server" not in _kept:
        _kept["serving"] = Benelux(device=0)
        _kept["server"] = Server(_kept["serving"], budget_bytes=8 << 30, max_inflight=2)
    return _kept["server"]


def listed():
    return [
        # The smallest search: one workgroup, all latency.
        {"name": "search_4k", "op": "search", "n": 4096, "kinds": 3},
        # A search of a few million integers, much of it below N/2 where small radicals count.
        {"name": "search_3m", "op": "search", "n": 3000017, "kinds": 3},
        # The whole-range searches of the published lists; the second is the headline workload.
        {"name": "search_2p32", "op": "search", "n": 1 << 32, "kinds": 3},
        {"name": "search_2p36", "op": "search", "n": 1 << 36, "kinds": 3},
        # Single range queries at the served trace's magnitude: its short, median and longest
        # lengths; with the third condition, with one kind, and with both kinds.
        {"name": "range_64k", "op": "range", "len": 65537, "kinds": 7},
        {"name": "range_1m", "op": "range", "len": 1 << 20, "kinds": 1},
        {"name": "range_256m", "op": "range", "len": 1 << 28, "kinds": 3},
        # The batched workload: thousands of queries of very different lengths.
        {"name": "batch_4096", "op": "batch", "count": 4096, "log2_min": 10, "log2_max": 24, "sizes": 2506, "kinds": 3},
        # Many short queries, each small enough for one workgroup.
        {"name": "batch_short_300", "op": "batch", "count": 300, "log2_min": 10, "log2_max": 13, "sizes": 7, "kinds": 3},
        # A burst of served requests, submitted together and collected as they finish.
        {"name": "served_48", "op": "served", "count": 48, "log2_min": 12, "log2_max": 26, "sizes": 1099, "kinds": 3},
        # Radicals into host memory (an odd length), and a large block left on the device.
        {"name": "radicals_host_300k", "op": "radicals", "where": "host", "len": 300007},
        {"name": "radicals_dev_200m", "op": "radicals", "where": "device", "len": 200000033},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["search", "search", "range", "range", "batch", "served", "radicals"])
    kinds = rng.choice([1, 2, 3, 3, 7])
    if op == "search":
        return {"op": op, "n": _log_uniform(rng, 1 << 10, 1 << 35), "kinds": kinds}
    if op == "range":
        return {"op": op, "len": _log_uniform(rng, 1 << 10, 1 << 28), "kinds": kinds}
    if op == "batch":
        lo = rng.randrange(8, 13)
        return {"op": op, "count": _log_uniform(rng, 8, 4096), "log2_min": lo, "log2_max": rng.randrange(lo + 1, 25),
                "sizes": rng.randrange(1, 1 << 20), "kinds": kinds}
    if op == "served":
        return {"op": op, "count": _log_uniform(rng, 4, 64), "log2_min": 12, "log2_max": rng.randrange(14, 29),
                "sizes": rng.randrange(1, 1 << 20), "kinds": kinds}
    if rng.random() < 0.5:
        return {"op": op, "where": "host", "len": _log_uniform(rng, 1 << 10, 1 << 22)}
    return {"op": op, "where": "device", "len": _log_uniform(rng, 1 << 10, 1 << 28)}


def _lengths(case):
    """The lengths of a batch's queries or a burst's requests, log-uniform."""
    rng = random.Random(case["sizes"])
    return [int(2.0 ** rng.uniform(case["log2_min"], case["log2_max"])) for _ in range(case["count"])]


def _where(case, seed):
    """The ranges [a, b) of the case: one, or one per query.  Most starts are uniform below
    2^40; every eighth query of a batch or burst starts among the first integers, where
    the pairs are (just past (35, 4374))."""
    rng = random.Random(1000003 * seed + 17)
    if case["op"] == "search":
        return [(1, case["n"] - rng.randrange(case["n"] // 64 + 1) + 1)]
    if case["op"] in ("batch", "served"):
        out = []
        for i, length in enumerate(_lengths(case)):
            a = 36 if i % 8 == 0 else rng.randrange(1, 1 << 40)
            out.append((a, a + length))
        return out
    a = rng.randrange(1 << 30, 1 << 40)
    return [(a, a + case["len"])]


def prepare(case, seed):
    ranges = _where(case, seed)
    state = {"op": case["op"], "a": ranges[0][0], "b": ranges[0][1], "kinds": case.get("kinds")}
    if case["op"] == "served":
        state["server"] = _server()
        state["requests"] = ranges
        return state
    state["ctx"] = _context()
    if case["op"] == "batch":
        state["starts"] = np.array([r[0] for r in ranges], dtype=np.uint64)
        state["ends"] = np.array([r[1] for r in ranges], dtype=np.uint64)
    if case["op"] == "radicals":
        state["where"] = case["where"]
        if case["where"] == "host":
            state["out"] = np.zeros(case["len"], dtype=np.uint64)
        else:
            state["out"] = torch.zeros(case["len"], dtype=torch.int64, device="cuda")
    return state


def _table(lists):
    """Pair lists of several ranges as one table: range number, m, n, kind."""
    rows = [(i, m, n, kind) for i, pairs in enumerate(lists) for m, n, kind in pairs]
    return np.array(rows, dtype=np.int64).reshape(-1, 4)


def _result(state, lists):
    """What a program files: the range, its pairs and the counts of the call."""
    st = state["ctx"].stats()
    return {"range": np.array([state["a"], state["b"]], dtype=np.int64), "pairs": _table(lists),
            "integers": st["integers"], "entries": st["entries"]}


def run(state):
    """One pass: the calls and their results (pair lists as tables, with the call's counts)."""
    if state["op"] == "served":
        server = state["server"]
        tickets = [server.submit(a, b, state["kinds"]) for a, b in state["requests"]]
        results = []
        for t in tickets:
            while not server.poll(t):
                pass
            results.append(server.take_pairs(t))
        return {"ranges": np.array(state["requests"], dtype=np.int64), "pairs": _table(results)}
    ctx = state["ctx"]
    if state["op"] == "search":
        return _result(state, [ctx.search(state["b"] - 1, state["kinds"])])
    if state["op"] == "range":
        return _result(state, [ctx.search_range(state["a"], state["b"], state["kinds"])])
    if state["op"] == "batch":
        return _result(state, ctx.search_batch(state["starts"], state["ends"], state["kinds"]))
    if state["where"] == "host":
        return ctx.radical_segment(state["a"], state["b"], state["out"])
    return ctx.radical_segment_dev(state["a"], state["b"], state["out"])


def work(case):
    """A search has to look at every integer (about 20 operations on 32-bit words each) and to
    bring together the 10.7% of them that can belong to a pair (8 bytes written and read
    once); radicals are written once, 8 bytes each."""
    if case["op"] == "radicals":
        return {"bytes": 8 * case["len"], "flops": 12 * case["len"]}
    if case["op"] in ("batch", "served"):
        n = sum(_lengths(case))
    else:
        n = case["n"] if case["op"] == "search" else case["len"]
    return {"bytes": int(0.107 * 16 * n), "flops": 20 * n}


def _pairs_inside(a, b, kinds):
    """Every pair a <= m < n < b (complete for n < 1.4e12): the two families and the two
    sporadic pairs of Theorem 1 of arXiv:2506.01099, as (m, n, kind)."""
    found = [(75, 1215, 1), (35, 4374, 2)]
    for k in range(2, 22):
        m = (1 << k) - 2
        found.append((m, (m << k), 1))
    for k in range(0, 22):
        m = (1 << k) + 1
        found.append((m, m * m - 1, 2))
    return sorted(p for p in set(found) if a <= p[0] and p[1] < b and (kinds & p[2]))


def _radicals(lo, hi):
    """rad(x) for lo <= x < hi: every multiple of p^k, k >= 2, divided once by p."""
    r = np.arange(lo, hi, dtype=np.int64)
    top = math.isqrt(hi)
    comp = np.zeros(top + 1, dtype=bool)
    for p in range(2, top + 1):
        if comp[p]:
            continue
        comp[p * p::p] = True
        q = p * p
        while q < hi:
            first = -lo % q
            if first < hi - lo:
                r[first::q] //= p
            q *= p
    return r


def exact(case, seed):
    ranges = _where(case, seed)
    if case["op"] == "radicals":
        if case["len"] > 1 << 23:
            return None
        r = _radicals(*ranges[0])
        return r.astype(np.uint64) if case["where"] == "host" else torch.from_numpy(r)
    pairs = _table([_pairs_inside(a, b, case["kinds"]) for a, b in ranges])
    if case["op"] == "served":
        return {"ranges": np.array(ranges, dtype=np.int64), "pairs": pairs}
    return {"range": np.array(ranges[0], dtype=np.int64), "pairs": pairs, "integers": sum(b - a for a, b in ranges),
            "entries": None}
