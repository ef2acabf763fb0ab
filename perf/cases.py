"""The work that a user of the table library has it do, as timed cases.

Each case is one call, or one short sequence of calls, through the Python
binding: lookups of one burst to a full-size batch on tables of 2^10 to 2^24
buckets, inserts and deletes from a burst's few keys to a whole build, tables
with timers, and many tables behind one plan.  Sizes follow the benchmark,
its serving and batching workloads and the tests.  Every input is drawn on
the GPU from the seed, in the form of network 5-tuples (two addresses, two
ports, protocol 6 or 17).

Every output is a whole number (found flags, values, statuses, counts), so
there is no rounding and no 64-bit reference to give.  The resident serving
loop is not here: its kernel holds every compute unit until it has been idle
for a while, so passes over several states would time that wait.
"""

from __future__ import annotations

import math

import torch

from paper_1712_09624_amd.ckpp import Plan, Table

HASH_SEED = 0x243F6A8885A308D3
NOW = 65000  # the 16-bit clock of the tables with timers (it wraps within the window)


def listed():
    return [
        # one burst of packets looked up as it arrives (the mean burst of the
        # latency benchmark): latency and one launch
        {"name": "burst_lookup", "op": "lookup", "log2_buckets": 24, "load": 0.85, "n": 269,
         "neg": 0.5, "mode": "cuckoopp"},
        # an ordinary batch on a table of the last-level cache's size, mostly
        # hits (the paper's multicore mix)
        {"name": "lookup_64k", "op": "lookup", "log2_buckets": 20, "load": 0.8, "n": 65536,
         "neg": 0.2, "mode": "cuckoopp"},
        # a large ragged batch on a small table (the parity workload's shape)
        {"name": "lookup_small_table", "op": "lookup", "log2_buckets": 14, "load": 0.8,
         "n": 1048573, "neg": 0.5, "mode": "cuckoopp"},
        # the benchmark step's two lookup batches: known flows, (nearly all) unknown flows
        {"name": "lookup_hits_64m", "op": "lookup", "log2_buckets": 24, "load": 0.9,
         "n": 1 << 26, "neg": 0.0, "mode": "cuckoopp"},
        {"name": "lookup_misses_64m", "op": "lookup", "log2_buckets": 24, "load": 0.9,
         "n": 1 << 26, "neg": 0.99, "mode": "cuckoopp"},
        # the plain table: no filter, both buckets read
        {"name": "lookup_plain_4m", "op": "lookup", "log2_buckets": 20, "load": 0.9,
         "n": 4000037, "neg": 0.25, "mode": "both"},
        # connection tracking: every hit renews its entry
        {"name": "lookup_renew_4m", "op": "renew", "log2_buckets": 22, "load": 0.9,
         "n": 1 << 22, "neg": 0.25},
        # many tables (one per tenant or port), one launch
        {"name": "plan_1024", "op": "plan", "tables": 1024, "log2_lo": 10, "log2_hi": 18,
         "batch_hi": 4096},
        # a serving burst through the plain calls: lookups, new flows, ended flows
        {"name": "burst_mixed", "op": "burst", "log2_buckets": 24, "load": 0.85, "n": 242,
         "updates": 27},
        # the benchmark step's churn: a batch of new flows in, an old one out
        {"name": "churn_64k", "op": "churn", "log2_buckets": 24, "load": 0.9, "n": 65536},
        # a table built to high load in one call and read back (32M slots)
        {"name": "build_32m", "op": "build", "log2_buckets": 22, "load": 0.95},
        # a table with timers over one period: new flows, the scan, ended flows
        {"name": "timed_churn_100k", "op": "timed_churn", "log2_buckets": 20, "load": 0.85,
         "n": 100003},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["lookup", "lookup", "lookup", "renew", "plan", "burst", "churn", "churn",
                     "build", "timed_churn"])
    load = round(rng.uniform(0.5, 0.95), 3)
    if op == "lookup":
        return {"op": op, "log2_buckets": rng.randint(10, 24), "load": load,
                "n": _log_int(rng, 8, 1 << 25), "neg": round(rng.random(), 3),
                "mode": rng.choice(["cuckoopp", "cuckoopp", "cuckoopp", "both", "optimistic"])}
    if op == "renew":
        return {"op": op, "log2_buckets": rng.randint(10, 23), "load": load,
                "n": _log_int(rng, 16, 1 << 23), "neg": round(rng.random(), 3)}
    if op == "plan":
        lo = rng.randint(8, 14)
        return {"op": op, "tables": _log_int(rng, 16, 1024), "log2_lo": lo,
                "log2_hi": lo + rng.randint(0, 4), "batch_hi": _log_int(rng, 64, 4096)}
    if op == "burst":
        n = _log_int(rng, 8, 2048)
        return {"op": op, "log2_buckets": rng.randint(16, 24), "load": round(min(load, 0.9), 3),
                "n": n, "updates": max(1, n // 9)}
    if op == "build":
        return {"op": op, "log2_buckets": rng.randint(10, 22), "load": load}
    b = rng.randint(14, 24) if op == "churn" else rng.randint(14, 22)
    # the batch fits beside the table's other entries (at most 0.95 in all)
    load = round(min(load, 0.9), 3)
    most = min(1 << 20, int(0.04 * (8 << b)))
    return {"op": op, "log2_buckets": b, "load": load, "n": _log_int(rng, 16, most)}


# ---- inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _keys(g, n):
    """n random 5-tuples (97 random bits each, so distinct) as (n, 16) bytes."""
    w = torch.randint(-(1 << 31), 1 << 31, (n, 4), dtype=torch.int32, device="cuda", generator=g)
    w[:, 3] = 6 + 11 * (w[:, 3] & 1)
    return w.view(torch.uint8).reshape(n, 16)


def _rows(keys):
    """Keys as rows of two 64-bit words, which torch indexes faster than bytes."""
    return keys.view(torch.int64)


def _take(keys, at):
    """Rows `at` of the keys; in parts, since torch launches a block per row."""
    return torch.cat([_rows(keys)[p] for p in at.split(1 << 24)])


def _mix(g, live, n, neg):
    """n lookups, each a random live key or (with probability neg) a fresh one."""
    fresh = torch.rand(n, 1, device="cuda", generator=g) < neg
    pick = torch.randint(0, live.shape[0], (n,), device="cuda", generator=g)
    rows = torch.where(fresh, _rows(_keys(g, n)), _take(live, pick))
    return rows.view(torch.uint8)


def _flows(g, live, n):
    """One batch of flows that come and go: the keys it inserts (one in ten is
    live already and only rewritten, with the value it has), their values, and
    the keys it later deletes (one in ten was never there)."""
    known = torch.rand(n, device="cuda", generator=g) < 0.1
    at = (int(torch.randint(0, live.shape[0], (1,), generator=g, device="cuda"))
          + torch.arange(n, device="cuda")) % live.shape[0]
    fresh, absent = _rows(_keys(g, n)), _rows(_keys(g, n))
    come = torch.where(known[:, None], _take(live, at), fresh).view(torch.uint8)
    go = torch.where(known[:, None], absent, fresh).view(torch.uint8)
    return {"come": come, "values": torch.where(known, at, _values(n)), "go": go}


def _count(case):
    return int(case["load"] * (8 << case["log2_buckets"]) + 0.5)


def _values(n):
    return torch.arange(n, dtype=torch.int64, device="cuda")


def _times(t):
    """16-bit times from a tensor of ints."""
    return (t & 0xFFFF).to(torch.int32).to(torch.int16)


def _outputs(n):
    return {"found": torch.empty(n, dtype=torch.uint8, device="cuda"),
            "values": torch.empty(n, dtype=torch.int64, device="cuda")}


def _timed_table(g, case):
    """A filled table with timers whose entries all outlive the case."""
    t = Table(case["log2_buckets"], HASH_SEED, timers=True)
    live = _keys(g, _count(case))
    ahead = torch.randint(100, 1024, (live.shape[0],), device="cuda", generator=g)
    t.insert_at(live, _values(live.shape[0]), _times(NOW + ahead), NOW)
    return t, live


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    if op == "lookup":
        t = Table(case["log2_buckets"], HASH_SEED, plain=case["mode"] == "both")
        live = _keys(g, _count(case))
        t.insert(live, _values(live.shape[0]))
        return {"op": op, "table": t, "mode": case["mode"],
                "keys": _mix(g, live, case["n"], case["neg"]), "out": _outputs(case["n"])}
    if op == "renew":
        t, live = _timed_table(g, case)
        return {"op": op, "table": t, "keys": _mix(g, live, case["n"], case["neg"]),
                "out": _outputs(case["n"]), "tick": 0}
    if op == "plan":
        return _prepare_plan(case, g)
    if op in ("burst", "churn"):
        # two sets of flows take turns: one is in the table, the other comes
        # in while it goes out, so every pass finds the table as full as before
        t = Table(case["log2_buckets"], HASH_SEED)
        n = case["updates"] if op == "burst" else case["n"]
        live = _keys(g, _count(case))
        sets = [_flows(g, live, n), _flows(g, live, n)]
        t.insert(live, _values(live.shape[0]))
        t.insert(sets[1]["come"], sets[1]["values"])
        s = {"op": op, "table": t, "sets": sets, "turn": 0}
        if op == "burst":
            s["keys"], s["out"] = _mix(g, live, case["n"], 0.1), _outputs(case["n"])
        return s
    if op == "build":
        n = _count(case)
        values = torch.randint(0, 1 << 62, (n,), device="cuda", generator=g)
        return {"op": op, "table": Table(case["log2_buckets"], HASH_SEED), "keys": _keys(g, n),
                "values": values, "out": _outputs(n)}
    # timed_churn: new flows, half of which expire before the scan
    t, _ = _timed_table(g, case)
    n = case["n"]
    ahead = torch.where(torch.rand(n, device="cuda", generator=g) < 0.5, 10, 1000)
    return {"op": op, "table": t, "keys": _keys(g, n), "values": _values(n),
            "times": _times(NOW + ahead)}


def _prepare_plan(case, g):
    n = case["tables"]
    u = torch.rand(4, n, generator=torch.Generator().manual_seed(n)).tolist()  # the fleet's sizes
    span = case["log2_hi"] - case["log2_lo"] + 1
    tables, offsets, counts, batches, at = [], [], [], [], 0
    for i in range(n):
        b = case["log2_lo"] + min(span - 1, int(u[0][i] * span))
        t = Table(b, HASH_SEED)
        live = _keys(g, int((0.6 + 0.35 * u[1][i]) * (8 << b)))
        t.insert(live, _values(live.shape[0]))
        c = 32 + int(u[2][i] * (case["batch_hi"] - 31))
        batches.append(_mix(g, live, c, u[3][i]))
        tables.append(t)
        offsets.append(at)
        counts.append(c)
        at += c
    return {"op": "plan", "plan": Plan(tables, offsets, counts), "keys": torch.cat(batches),
            "out": _outputs(at)}


# ---- one pass


def run(state):
    op, out = state["op"], state.get("out")
    if op == "plan":
        return state["plan"].lookup(state["keys"], out["found"], out["values"])
    t = state["table"]
    if op == "lookup":
        return t.lookup(state["keys"], state["mode"], found=out["found"], values=out["values"])
    if op == "renew":
        # the renewed time moves with the clock: each pass writes every hit's time
        state["tick"] ^= 1
        return t.lookup_at(state["keys"], NOW, refresh=NOW + 900 + state["tick"],
                           found=out["found"], values=out["values"])
    if op in ("burst", "churn"):
        new, old = state["sets"][state["turn"]], state["sets"][1 - state["turn"]]
        state["turn"] ^= 1
        got = []
        if op == "burst":
            got += t.lookup(state["keys"], found=out["found"], values=out["values"])
        got += t.insert(new["come"], new["values"])
        got.append(t.delete(old["go"]))
        return got
    if op == "build":
        t.clear()
        got = list(t.insert(state["keys"], state["values"]))
        return got + list(t.lookup(state["keys"], found=out["found"], values=out["values"]))
    got = list(t.insert_at(state["keys"], state["values"], state["times"], NOW))
    got.append(t.expire_scan(NOW + 50))
    got.append(t.delete_at(state["keys"], NOW + 50))
    return got


# ---- what a pass cannot do without

# A bucket's metadata in the paper's layout is one 64-byte line; an entry is a
# 16-byte key and an 8-byte value.  Streams: 16 bytes of key in, a byte of
# found and 8 bytes of value out per lookup; 16 + 8 in and a byte out per
# insert; 16 in and a byte out per delete.
_LINE, _ENTRY = 64, 24


def _lookup_bytes(n, neg, lines=1.0):
    return n * (25 + _LINE * lines + _ENTRY * (1.0 - neg))


def _insert_bytes(n):
    return n * (25 + 2 * _LINE + _ENTRY)


def _delete_bytes(n):
    return n * (17 + 2 * _LINE + 16)


def work(case):
    op = case["op"]
    slots = 8 << case["log2_buckets"] if "log2_buckets" in case else 0
    if op == "lookup":
        lines = {"cuckoopp": 1.0, "both": 2.0, "optimistic": 1.0 + case["neg"]}[case["mode"]]
        b = _lookup_bytes(case["n"], case["neg"], lines)
    elif op == "renew":
        b = _lookup_bytes(case["n"], case["neg"]) + case["n"] * (1 - case["neg"]) * 2
    elif op == "plan":
        b = _lookup_bytes(case["tables"] * (32 + case["batch_hi"]) / 2, 0.5)
    elif op == "burst":
        u = case["updates"]
        b = _lookup_bytes(case["n"], 0.1) + _insert_bytes(u) + _delete_bytes(u)
    elif op == "churn":
        b = _insert_bytes(case["n"]) + _delete_bytes(case["n"])
    elif op == "build":
        # every bucket's metadata and entries written once, then read back
        n = _count(case)
        b = 24 * n + 32 * slots + n + _lookup_bytes(n, 0.0)
    else:
        # the scan reads every entry's time beside its bucket's metadata
        b = (_insert_bytes(case["n"]) + _delete_bytes(case["n"]) + 2 * case["n"]
             + slots * (_LINE / 8 + 2))
    return {"bytes": float(b), "flops": 0.0}
