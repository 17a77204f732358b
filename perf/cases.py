"""Workloads of the library's public entry points, each at a size and on values that users run it with.

A case is a dict of plain values whose "kind" names the call:

  join         join_plain: build + probe, aggregates; with "rows" also build() and probe_rows()
  star         join_star: filtered dimensions, one fact table, GROUP BY
  batch        join_batch: many independent joins in one call
  partition    partition: stable clustering of a key column and its payload by partition
  partitioned  join_partitioned: a skewed build side, clustered, and one stream of the probe side
  radix        join_radix: the two-table radix-partitioned join
  sort         sort: a key column in place, in one run or out of core

"where" says where the big columns live: "device", or "host" (pinned memory that the library streams).
"""
import math

import numpy as np
import torch

import paper_2502_09541_amd as vx

MIB = 1 << 20
TYPES = {"i32": torch.int32, "i64": torch.int64}
GROUP_DIMS = (7, None, None, 100)   # group attribute values per dimension (None: no group attribute)
DIM_FILTERS = (7, 5, 25, 1)         # a dimension row passes its filter with probability 1 / this


def listed():
    return [
        # a lookup join of a small dimension, where launches and round trips are the whole cost
        dict(name="join_small", kind="join", where="device", key="i32", keys="dense", build=1000, probe=10007,
             build_pays="i32", probe_pays="", hit=0.5, unique=True, rows=False, budget_mib=64),
        # the in-memory join of the benchmark: 2^20 surrogate keys, 2^24 probe rows
        dict(name="join_memory", kind="join", where="device", key="i32", keys="dense", build=1 << 20, probe=1 << 24,
             build_pays="i32", probe_pays="", hit=0.5, unique=True, rows=False, budget_mib=1024),
        # natural 64-bit keys (hash table), payloads on both sides, odd row counts
        dict(name="join_hashed", kind="join", where="device", key="i64", keys="sparse", build=1500007, probe=12000017,
             build_pays="i32,i32", probe_pays="i64", hit=0.5, unique=True, rows=False, budget_mib=1024),
        # a build side with repeated keys: about four rows a key
        dict(name="join_duplicates", kind="join", where="device", key="i64", keys="sparse", build=3000017,
             probe=12000017, build_pays="i64", probe_pays="", hit=0.5, unique=False, rows=False, budget_mib=1024),
        # the streamed join of the benchmark, shortened: columns in pinned memory, 10% of the probe rows match
        dict(name="join_streamed", kind="join", where="host", key="i64", keys="sparse", build=1 << 20,
             probe=(1 << 24) + 77, build_pays="i32,i32", probe_pays="i64,i64", hit=0.1, unique=True, rows=False,
             budget_mib=1024),
        # a star query: four filtered dimensions on the GPU, the fact table in pinned memory, 700 groups
        dict(name="star", kind="star", where="host", dim0=2556, dim1=20000, dim2=300000, dim3=200000, fact=12000007,
             measures=3, budget_mib=1024),
        # a batch of device-resident joins of mixed sizes
        dict(name="batch", kind="batch", jobs=64, build_lo=1 << 10, build_hi=1 << 20, ratio_lo=10, ratio_hi=100,
             budget_mib=4096),
        # clustering a table (8-byte key, 8-byte payload) into 256 hash partitions on the device
        dict(name="partition", kind="partition", where="device", key="i64", method="radix_hash", parts=256,
             rows=16000007, pay="i64", budget_mib=1024),
        # the skewed partitioned join of the benchmark, shortened: Zipf keys, method chosen from the sample
        dict(name="join_partitioned", kind="partitioned", where="host", method="auto", parts=256, build=8000009,
             probe=32000011, budget_mib=1024),
        # the two-table join of the benchmark, shortened: 16-byte tuples, a table larger than the budget
        dict(name="join_radix", kind="radix", where="host", a=(1 << 24) + 5, b=(1 << 24) + 11, budget_mib=1024),
        # sorting a device column that fits the arena
        dict(name="sort_device", kind="sort", where="device", key="i64", rows=16000033, budget_mib=1024),
        # the out-of-core sort of the benchmark, shortened: eight runs through a small arena
        dict(name="sort_out_of_core", kind="sort", where="host", key="i64", rows=(1 << 24) - 3, budget_mib=128),
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], log-uniform, odd as often as even."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["join", "join", "join", "star", "batch", "partition", "partitioned", "radix", "sort", "sort"])
    if kind == "join":
        build = _log(rng, 1 << 10, 1 << 21)
        unique = rng.random() < 0.75
        pays = lambda least: ",".join(rng.choice(["i32", "i64"]) for _ in range(rng.randint(least, 2)))  # noqa: E731
        return dict(kind="join", where=rng.choice(["device", "device", "host"]), key=rng.choice(["i32", "i64"]),
                    keys=rng.choice(["dense", "sparse"]), build=build,
                    probe=min(1 << 24, int(build * math.exp(rng.uniform(0, math.log(64))))), build_pays=pays(1),
                    probe_pays=pays(0), hit=rng.choice([0.1, 0.5, 0.9]), unique=unique,
                    rows=unique and rng.random() < 0.3, budget_mib=1024)
    if kind == "star":
        fact = _log(rng, 1 << 18, 12000000)
        return dict(kind="star", where=rng.choice(["device", "host"]), dim0=_log(rng, 300, 3000),
                    dim1=_log(rng, 2000, 20000), dim2=_log(rng, 20000, 300000), dim3=_log(rng, 10000, 200000),
                    fact=fact, measures=rng.randint(1, 4), budget_mib=1024)
    if kind == "batch":
        return dict(kind="batch", jobs=rng.randint(4, 64), build_lo=1 << 10, build_hi=_log(rng, 1 << 13, 1 << 20),
                    ratio_lo=5, ratio_hi=rng.randint(10, 60), budget_mib=4096)
    if kind == "partition":
        method = rng.choice(["radix_hash", "radix_hash", "radix_bits", "quantile"])
        sampled = method == "quantile"
        return dict(kind="partition", where=rng.choice(["device", "device", "host"]), key=rng.choice(["i32", "i64"]),
                    method=method, parts=rng.choice([4, 16, 64] if sampled else [4, 16, 64, 256, 1024]),
                    rows=_log(rng, 1 << (20 if sampled else 16), 16000000), pay=rng.choice(["", "i32", "i64"]),
                    budget_mib=1024)
    if kind == "partitioned":
        build = _log(rng, 1 << 18, 8000000)
        return dict(kind="partitioned", where=rng.choice(["device", "host"]),
                    method=rng.choice(["auto", "quantile", "radix_hash"]), parts=rng.choice([64, 256]), build=build,
                    probe=build * rng.randint(2, 4) + rng.randint(0, 99), budget_mib=2048)
    if kind == "radix":
        return dict(kind="radix", where=rng.choice(["device", "host"]), a=_log(rng, 1 << 18, 1 << 24),
                    b=_log(rng, 1 << 18, 1 << 24), budget_mib=rng.choice([768, 1024, 4096]))
    rows = _log(rng, 1 << 12, 16000000)
    where = rng.choice(["device", "device", "host"])
    return dict(kind="sort", where=where, key=rng.choice(["i32", "i64"]), rows=rows,
                budget_mib=1024 if where == "device" else max(16, rows * 8 // MIB))


# ---------------------------------------------------------------------------- inputs

class _Random:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def ints(self, lo, hi, n, dtype=torch.int64):
        return torch.randint(lo, hi, (n,), generator=self.g, device="cuda", dtype=dtype)

    def unit(self, n):
        return torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64)

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device="cuda")

    def payload(self, n, t):
        return self.ints(-(1 << 31), 1 << 31, n, torch.int32) if t == "i32" else self.ints(-(1 << 32), 1 << 32, n)


def _spread(i, key):
    """A bijection that scatters row numbers over [0, 2^40) (64-bit keys) or all 32-bit values."""
    bits, half = (40, 20) if key == "i64" else (32, 16)
    mask = (1 << bits) - 1
    i = (i * 0x1E3779B97F4A7C15) & mask
    i = i ^ (i >> half)
    i = (i * 0x42B2AE3D27D4EB4F) & mask
    i = i ^ (i >> half)
    return i if key == "i64" else (i - (1 << 31)).to(torch.int32)


def _keys(i, case):
    return i.to(TYPES[case["key"]]) if case["keys"] == "dense" else _spread(i, case["key"])


def _zipf(r, n):
    """Ranks of a power law with exponent 1.1 over [1, 2^40] (the continuous law, rounded down)."""
    top = float(1 << 40) ** -0.1
    return (1.0 + r.unit(n) * (top - 1.0)).pow(-10.0).floor().to(torch.int64).clamp_(1, 1 << 40)


def _types(text):
    return [t for t in text.split(",") if t]


def _columns(case, seed):
    """The case's columns as device tensors, by name; lists where a call takes lists."""
    r, kind = _Random(seed), case["kind"]
    if kind == "join":
        nb, n = case["build"], case["probe"]
        if case["unique"]:
            bi, most = r.perm(nb), nb
        else:
            most = max(1, nb // 4)
            bi = r.ints(0, most, nb)
        pi = r.ints(0, most, n)
        pi = torch.where(r.perm(n) < int(n * case["hit"]), pi, pi + most)
        return dict(bkey=_keys(bi, case), bpays=[r.payload(nb, t) for t in _types(case["build_pays"])],
                    pkey=_keys(pi, case), ppays=[r.payload(n, t) for t in _types(case["probe_pays"])])
    if kind == "star":
        rows = [case["dim%d" % d] for d in range(4)]
        dims = [dict(key=torch.arange(m, device="cuda", dtype=torch.int32), filt=r.ints(0, q, m, torch.int32), lo=0,
                     hi=0, group=None if g is None else r.ints(0, g, m, torch.int32))
                for m, q, g in zip(rows, DIM_FILTERS, GROUP_DIMS)]
        return dict(dims=dims, fks=[r.ints(0, m, case["fact"], torch.int32) for m in rows],
                    meas=[r.ints(0, 1 << 20, case["fact"], torch.int32) for _ in range(case["measures"])])
    if kind == "batch":
        c = dict(bkeys=[], bpays=[], pkeys=[])
        u = r.unit(2 * case["jobs"]).cpu().tolist()
        for j in range(case["jobs"]):
            nb = int(case["build_lo"] * (case["build_hi"] / case["build_lo"]) ** u[2 * j])
            n = int(nb * case["ratio_lo"] * (case["ratio_hi"] / case["ratio_lo"]) ** u[2 * j + 1])
            c["bkeys"].append(r.perm(nb).to(torch.int32))
            c["bpays"].append(r.payload(nb, "i32"))
            c["pkeys"].append(r.ints(0, 2 * nb, n, torch.int32))
        return c
    if kind == "partition":
        n = case["rows"]
        return dict(key=_spread(r.ints(0, max(2, n // 2), n), case["key"]),
                    pays=[r.payload(n, t) for t in _types(case["pay"])])
    if kind == "partitioned":
        return dict(bkey=_zipf(r, case["build"]), bpays=[r.ints(0, 1 << 32, case["build"])],
                    pkey=_zipf(r, case["probe"]))
    if kind == "radix":
        return dict(akey=r.perm(case["a"]), apays=[r.ints(0, 1 << 32, case["a"])],
                    bkey=r.ints(0, case["a"], case["b"]), bpays=[r.ints(0, 1 << 32, case["b"])])
    if case["key"] == "i64":
        return dict(key=r.ints(-(1 << 63), (1 << 63) - 1, case["rows"]))
    return dict(key=r.ints(-(1 << 31), 1 << 31, case["rows"], torch.int32))


def _pinned(x):
    return torch.empty(x.shape, dtype=x.dtype, pin_memory=True).copy_(x)


def prepare(case, seed):
    s, kind = _columns(case, seed), case["kind"]
    if kind == "partition":
        s["out_key"] = torch.empty_like(s["key"])
        s["out_pays"] = [torch.empty_like(p) for p in s["pays"]]
    if kind == "join" and case["rows"]:
        cap = max(1, int(case["probe"] * case["hit"]))   # room for every matching row
        blank = lambda: torch.zeros(cap, dtype=torch.int64, device="cuda")  # noqa: E731
        s["out"] = (blank(), [blank() for _ in s["bpays"]], [blank() for _ in s["ppays"]])
    if kind == "sort":
        # each pass sorts a freshly arrived column: the unsorted keys are kept beside it
        s["column"] = _pinned(s["key"]) if case["where"] == "host" else torch.empty_like(s["key"])
    elif case.get("where") == "host":
        for k in ("bkey", "pkey", "akey", "key"):
            if k in s:
                s[k] = _pinned(s[k])
        for k in ("bpays", "ppays", "apays", "pays", "fks", "meas"):
            if k in s:
                s[k] = [_pinned(x) for x in s[k]]
    s["case"] = case
    s["ctx"] = vx.Context(case["budget_mib"] * MIB)
    return s


# ---------------------------------------------------------------------------- one pass

def _words(v):
    """Sums mod 2^64 as signed 64-bit words."""
    return np.array(v, dtype=np.uint64).view(np.int64)


def _report(*columns):
    """Group rows in a report of one line for every group there can be; short inputs leave some empty."""
    out = [np.zeros((GROUP_DIMS[0] * GROUP_DIMS[3],) + c.shape[1:], dtype=np.int64) for c in columns]
    for o, c in zip(out, columns):
        o[:len(c)] = c
    return out


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "join":
        if case["rows"]:
            table = ctx.build(s["bkey"], s["bpays"])
            agg, _, n, out = table.probe_rows(s["pkey"], s["ppays"], out=s["out"])
            table.destroy()
            # the rows come in no particular order: brought into the probe's order, as a reader would
            row, order = torch.sort(out[0][:n])
            return _words(agg), row, [c[:n][order] for c in out[1]], [c[:n][order] for c in out[2]]
        return _words(ctx.join_plain(s["bkey"], s["bpays"], s["pkey"], s["ppays"], unique=case["unique"])[0])
    if kind == "star":
        groups, count, sums, _ = ctx.join_star(s["dims"], s["fks"], s["meas"])
        return _report(groups, count.view(np.int64), sums.view(np.int64))
    if kind == "batch":
        return _words(ctx.join_batch(s["bkeys"], s["bpays"], s["pkeys"])[0])
    if kind == "partition":
        got = ctx.partition(s["key"], s["pays"], method=case["method"], n_parts=case["parts"], out_key=s["out_key"],
                            out_pays=s["out_pays"], seed=1)
        return got["hist"].view(np.int64), got["boundary"].view(np.int64), s["out_key"], s["out_pays"]
    if kind == "partitioned":
        return _words(ctx.join_partitioned(s["bkey"], s["bpays"], s["pkey"], method=case["method"],
                                           n_parts=case["parts"], seed=1)[0])
    if kind == "radix":
        return _words(ctx.join_radix(s["akey"], s["apays"], s["bkey"], s["bpays"])[0])
    s["column"].copy_(s["key"])
    ctx.sort(s["column"])
    return s["column"]


# ---------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Inputs read once and outputs written once; payload columns of the probe side only where a row matches."""
    kind, size = case["kind"], {"i32": 4, "i64": 8}
    if kind == "join":
        ks, bp, pp = size[case["key"]], _types(case["build_pays"]), _types(case["probe_pays"])
        match = case["probe"] * case["hit"]
        b = case["build"] * (ks + sum(size[t] for t in bp)) + case["probe"] * ks + match * sum(size[t] for t in pp)
        if case["rows"]:
            b += match * 8 * (1 + len(bp) + len(pp))
        return {"bytes": b, "flops": case["build"] + case["probe"]}
    if kind == "star":
        sel = [1.0 / q for q in sorted(DIM_FILTERS, reverse=True)]
        alive = [1.0, sel[0], sel[0] * sel[1], sel[0] * sel[1] * sel[2]]
        per = 4 * sum(alive) + 4 * case["measures"] * alive[3] * sel[3]
        dims = sum(case["dim%d" % d] * (8 if g is None else 12) for d, g in enumerate(GROUP_DIMS))
        return {"bytes": dims + per * case["fact"], "flops": case["fact"] * sum(alive)}
    if kind == "batch":
        mean = lambda lo, hi: (hi - lo) / math.log(hi / lo)  # noqa: E731
        nb = case["jobs"] * mean(case["build_lo"], case["build_hi"])
        n = nb * mean(case["ratio_lo"], case["ratio_hi"])
        return {"bytes": 8 * nb + 4 * n, "flops": nb + n}
    if kind == "partition":
        row = size[case["key"]] + size.get(case["pay"], 0)
        return {"bytes": 2 * row * case["rows"], "flops": case["rows"]}
    if kind == "partitioned":
        return {"bytes": 16 * case["build"] + 8 * case["probe"], "flops": case["build"] + case["probe"]}
    if kind == "radix":
        return {"bytes": 16 * (case["a"] + case["b"]), "flops": case["a"] + case["b"]}
    # the unsorted column is copied in (read, write), then sorted (read, write)
    return {"bytes": 4 * size[case["key"]] * case["rows"], "flops": case["rows"] * math.log2(case["rows"])}


# ---------------------------------------------------------------------------- the same from torch alone

def _grouped(key, *columns):
    """Distinct keys, their row counts and the sum of each column per key."""
    uniq, at = torch.unique(key, return_inverse=True)
    zero = lambda: torch.zeros(uniq.numel(), dtype=torch.int64, device="cuda")  # noqa: E731
    ones = torch.ones(key.numel(), dtype=torch.int64, device="cuda")
    return [uniq, zero().index_add_(0, at, ones)] + [zero().index_add_(0, at, c.long()) for c in columns]


def _lookup(uniq, key):
    """The position of every key in `uniq`, and whether it is there."""
    at = torch.searchsorted(uniq, key).clamp_(max=uniq.numel() - 1)
    return at, uniq[at] == key


def _agg(bkey, bpays, pkey, ppays):
    uniq, count, *sums = _grouped(bkey, *bpays)
    at, hit = _lookup(uniq, pkey)
    at = at[hit]
    mult = count[at]
    out = [mult.sum()] + [x[at].sum() for x in sums] + [(p.long()[hit] * mult).sum() for p in ppays]
    return np.array([int(v) for v in out], dtype=np.int64)


def _hash64(k):
    """MurmurHash3's 64-bit finalizer (Appleby, public domain), on the two's complement bits."""
    signed = lambda v: v - (1 << 64) if v >> 63 else v  # noqa: E731
    for mult in (0xFF51AFD7ED558CCD, 0xC4CEB9FE1A85EC53):
        k = (k ^ ((k >> 33) & ((1 << 31) - 1))) * signed(mult)
    return k ^ ((k >> 33) & ((1 << 31) - 1))


def exact(case, seed):
    c, kind = _columns(case, seed), case["kind"]
    if kind == "join":
        agg = _agg(c["bkey"], c["bpays"], c["pkey"], c["ppays"])
        if not case["rows"]:
            return agg
        order = torch.argsort(c["bkey"])
        at, hit = _lookup(c["bkey"][order], c["pkey"])
        row = torch.nonzero(hit).flatten()
        return agg, row, [p.long()[order][at[row]] for p in c["bpays"]], [p.long()[row] for p in c["ppays"]]
    if kind == "star":
        alive = torch.ones(case["fact"], dtype=torch.bool, device="cuda")
        for d, fk in zip(c["dims"], c["fks"]):
            alive &= (d["filt"] == 0)[fk.long()]
        g = [d["group"][fk.long()][alive].long() for d, fk in zip(c["dims"], c["fks"]) if d["group"] is not None]
        uniq, count, *sums = _grouped(g[0] << 32 | g[1], *[m[alive] for m in c["meas"]])
        groups = torch.stack([uniq >> 32, uniq & 0xFFFFFFFF], 1)
        return _report(groups.cpu().numpy(), count.cpu().numpy(), torch.stack(sums, 1).cpu().numpy())
    if kind == "batch":
        return np.stack([_agg(b, [p], k, []) for b, p, k in zip(c["bkeys"], c["bpays"], c["pkeys"])])
    if kind == "partition":
        bits = case["parts"].bit_length() - 1
        key = c["key"].long()
        if case["method"] == "radix_hash":
            part = (_hash64(key) >> (64 - bits)) & (case["parts"] - 1)
        elif case["method"] == "radix_bits":
            part = key & (case["parts"] - 1)
        else:
            return None   # splitters drawn from a sample of the keys have no value of their own
        order = torch.argsort(part, stable=True)
        hist = torch.bincount(part, minlength=case["parts"])
        boundary = torch.cat([hist.new_zeros(1), hist.cumsum(0)])
        return hist.cpu().numpy(), boundary.cpu().numpy(), c["key"][order], [p[order] for p in c["pays"]]
    if kind == "partitioned":
        return _agg(c["bkey"], c["bpays"], c["pkey"], [])
    if kind == "radix":
        return _agg(c["akey"], c["apays"], c["bkey"], c["bpays"])
    return torch.sort(c["key"])[0]
