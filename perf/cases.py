"""What a program built on the embedding cache has it do: one case per kind of call sequence and size.

A case is a dict of plain values; `prepare` builds what the program holds before the call (cache,
key batches, result buffers), `run` is one pass through the public entry points of
paper_2210_08804_amd.binding, `exact` states the same result in plain torch.

Batches follow the serving workloads of the repository's benchmark: samples x 26 categorical
features, power-law key popularity, rows of 16 to 512 fp32, most of a query's keys cached.  Every
state holds several batches and a pass takes the next one, as a server sees a new batch with every
request.  Which keys are cached is a function of the seed alone: the resident keys asked for are
chosen so that no set gets more of them than it has ways, and they are inserted last.

Miss lists have no particular order, so they are not returned; the cases that fill missing rows
consume them, and a wrong entry there is a wrong row of `out`.  Likewise the way in which an insert
distributes one batch over the slots of a set is free; the rows read back afterwards are not.
"""
import math

import numpy as np
import torch

from paper_2210_08804_amd import binding as B

FEATURES = 26
OPS = ("query", "multi", "stream", "publish", "refresh", "dedup", "lookup")


def listed():
    return [
        # the smallest request: 32 samples, default mode (rows validated against concurrent writers)
        dict(name="query_32_samples", op="query", keys=32 * FEATURES, sets=1 << 18, ways=8, dim=128, policy="counter", checked=True),
        # an ordinary serving batch of 1024 samples on a cache with the LRU policy, default mode
        dict(name="query_1024_samples_lru", op="query", keys=1024 * FEATURES, sets=1 << 19, ways=8, dim=128, policy="lru", checked=True),
        # the benchmark's batch against its 8 GiB hot cache, no writer overlapping
        dict(name="query_4096_samples", op="query", keys=4096 * FEATURES, sets=1 << 21, ways=8, dim=128, policy="counter", checked=False),
        # the same batch in the default mode
        dict(name="query_4096_samples_default", op="query", keys=4096 * FEATURES, sets=1 << 20, ways=8, dim=128, policy="counter", checked=True),
        # a large batch of short rows, default mode
        dict(name="query_32768_samples_d32", op="query", keys=32768 * FEATURES, sets=1 << 20, ways=8, dim=32, policy="counter", checked=True),
        # a ragged batch of long rows, set count not a power of two
        dict(name="query_ragged_d320", op="query", keys=39999, sets=100003, ways=8, dim=320, policy="counter", checked=False),
        # one table per categorical feature, a large batch in one call
        dict(name="multi_26_tables", op="multi", tables=FEATURES, keys=65536, sets=1 << 14, ways=8, dim=128, checked=False),
        # query, fetch of the missing rows, insert of them, on a cache much smaller than the key space
        dict(name="stream_16384_samples", op="stream", keys=16384 * FEATURES, sets=1 << 16, ways=8, dim=128, policy="counter", checked=False),
        # a batch of new embeddings: inserted, then updated by a newer version, then served
        dict(name="publish_262144_rows", op="publish", keys=1 << 18, sets=1 << 20, ways=8, dim=128, policy="counter", checked=True),
        # whole-cache refresh of 1 GiB of rows: dump, update, one serving batch
        dict(name="refresh_1gib", op="refresh", keys=4096 * FEATURES, sets=1 << 18, ways=8, dim=128, checked=True),
        # the deduplicated lookup: distinct keys, their query, fetch of the missing ones, expansion
        dict(name="dedup_4096_samples", op="dedup", keys=4096 * FEATURES, sets=1 << 20, ways=8, dim=128, policy="counter", checked=True),
        # Algorithm 1 with synchronous insertion, the library's host map as the lower tier
        dict(name="lookup_1024_samples", op="lookup", keys=1024 * FEATURES, sets=1638, ways=8, dim=128, policy="lru", space=1 << 18),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  Its row traffic stays below that of the largest listed one."""
    op = rng.choices(OPS, weights=(6, 1, 2, 2, 1, 2, 1))[0]
    dim = rng.choice((16, 32, 64, 96, 100, 128, 128, 128, 192, 256, 320, 512))
    ways = rng.choice((4, 8, 8, 8, 16))
    c = dict(op=op, dim=dim, ways=ways)
    row_cap = (1 << 26) // dim                     # rows moved by one pass
    slot_cap = (1 << 28) // dim                    # rows cached
    if op == "query":
        c["keys"] = min(_log_uniform(rng, 64, 32768 * FEATURES), row_cap)
        c["sets"] = min(_log_uniform(rng, 1 << 13, 1 << 20), slot_cap // ways)
        c["policy"] = rng.choice(("counter", "counter", "lru"))
        c["checked"] = rng.random() < 0.6
    elif op == "multi":
        c["tables"] = rng.randint(2, FEATURES)
        c["keys"] = max(16, min(_log_uniform(rng, 32, 65536), row_cap // c["tables"]))
        c["sets"] = min(_log_uniform(rng, 1 << 10, 1 << 14), slot_cap // (ways * c["tables"]))
        c["checked"] = rng.random() < 0.5
    elif op == "stream":
        c["keys"] = min(_log_uniform(rng, 832, 16384 * FEATURES), row_cap // 4)
        c["sets"] = max(256, min(c["keys"] // 4 + rng.randint(0, 99), slot_cap // ways))
        c["policy"] = rng.choice(("counter", "counter", "lru"))
        c["checked"] = rng.random() < 0.5
    elif op == "publish":
        c["ways"] = max(8, ways)
        c["keys"] = min(_log_uniform(rng, 256, 1 << 18), row_cap // 6)
        c["sets"] = max(4096, min(8 * c["keys"] + rng.randint(0, 99), slot_cap // c["ways"]))
        c["policy"] = rng.choice(("counter", "counter", "lru"))
        c["checked"] = rng.random() < 0.5
        c["keys"] = min(c["keys"], c["sets"] // 4)
    elif op == "refresh":
        c["sets"] = min(_log_uniform(rng, 1 << 12, 1 << 18), slot_cap // ways)
        c["keys"] = min(_log_uniform(rng, 832, 4096 * FEATURES), row_cap // 4)
        c["checked"] = rng.random() < 0.5
    elif op == "dedup":
        c["keys"] = min(_log_uniform(rng, 832, 16384 * FEATURES), row_cap // 2)
        c["sets"] = min(_log_uniform(rng, 1 << 13, 1 << 19), slot_cap // ways)
        c["policy"] = "counter"
        c["checked"] = rng.random() < 0.5
    else:
        c["keys"] = min(_log_uniform(rng, 832, 1024 * FEATURES), row_cap // 16)
        c["space"] = min(_log_uniform(rng, 1 << 14, 1 << 18), (1 << 25) // dim)
        c["sets"] = max(64, c["space"] // (20 * ways))
        c["policy"] = rng.choice(("counter", "lru"))
    return c


# ---- keys and rows, in plain torch ------------------------------------------------------------

ALPHA = 1.05
HIT = 0.93                                         # share of a query's positions whose key is cached
_COLD, _ABSENT = 1 << 40, 1 << 41                  # id ranges: cached but never asked for; never cached


def _shr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _mix(x):
    """splitmix64 finaliser on int64 tensors (wrapping products)."""
    x = (x ^ _shr(x, 30)) * (0xBF58476D1CE4E5B9 - (1 << 64))
    x = (x ^ _shr(x, 27)) * (0x94D049BB133111EB - (1 << 64))
    return x ^ _shr(x, 31)


def _rows(keys, dim, version=0):
    """The row a lower tier holds for each key: the definition of hps_backing_fetch, as float32."""
    j = torch.arange(dim, dtype=torch.int64, device="cuda") | (version << 32)
    inner = _mix(j + (0x9E3779B97F4A7C15 - (1 << 64)))
    out = torch.empty(len(keys), dim, dtype=torch.float32, device="cuda")
    for lo in range(0, len(keys), 1 << 18):
        z = _shr(_mix(keys[lo:lo + (1 << 18), None] ^ inner[None, :]), 40) - (1 << 23)
        out[lo:lo + (1 << 18)] = z.to(torch.float32) * 2.0 ** -23
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _base(seed):
    """First id of a seed's key ranges: other seeds have other keys."""
    return (seed * 0x9E3779B1 + 12345) % (1 << 20) << 42


def _zipf(n, space, alpha, g):
    """n ranks in [0, space), p(r) about (r + 1)^-alpha."""
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=g)
    a = 1.0 - alpha
    r = torch.floor((1.0 + u * (float(space) ** a - 1.0)) ** (1.0 / a))
    return r.clamp_(1.0, float(space)).to(torch.int64) - 1


def _resident(sets, ways, seed):
    """Keys that a cache of this geometry can hold all at once: about half its slots, most popular first."""
    keys = _base(seed) + torch.arange(sets * ways // 2, dtype=torch.int64, device="cuda")
    where = _shr(_mix(keys), 32) % sets
    order = torch.argsort(where, stable=True)
    s = where[order]
    first = torch.searchsorted(s, s)               # start of the key's set in the sorted list
    keep = torch.zeros(len(keys), dtype=torch.bool, device="cuda")
    keep[order] = torch.arange(len(keys), device="cuda") - first < ways
    return keys[keep]


def _batches(n, resident, seed, count):
    """`count` batches of n keys: power-law over the resident keys, the rest over keys that are nowhere."""
    g = _generator(seed)
    keys = resident[_zipf(n * count, len(resident), ALPHA, g)]
    missing = _base(seed) + _ABSENT + _zipf(n * count, 1 << 30, ALPHA, g)
    hit = torch.rand(n * count, device="cuda", generator=g) < HIT
    return torch.where(hit, keys, missing).view(count, n), hit.view(count, n)


def _turns(n):
    return max(4, min(128, (1 << 22) // n))


def _stream_space(case):
    return 64 * case["sets"] * case["ways"]


# ---- state ------------------------------------------------------------------------------------

class _State:
    """Handles and buffers of one program; the handles go back when the state does."""

    def __init__(self, case):
        self.case = case
        self.closers = []
        self.turn = 0

    def cache(self, sets, ways, dim, policy="counter"):
        h = B.hps_cache_create_policy(sets * ways, ways, dim, B.HPS_POLICY_LRU if policy == "lru" else B.HPS_POLICY_VICTIM_COUNTER)
        self.closers.append(lambda: B.hps_cache_destroy(h))
        return h

    def result(self, n, dim):
        self.out = torch.zeros(n, dim, dtype=torch.float32, device="cuda")
        self.miss_idx = torch.zeros(n, dtype=torch.int32, device="cuda")
        self.miss_keys = torch.zeros(n, dtype=torch.int64, device="cuda")
        self.n_miss = torch.zeros(1, dtype=torch.int32, device="cuda")

    def next(self):
        t = self.turn
        self.turn = t + 1
        return self.keys[t % len(self.keys)]

    def __del__(self):
        if self.closers:
            torch.cuda.synchronize()
        while self.closers:
            self.closers.pop()()


def _fill(h, sets, ways, dim, resident, seed):
    """Cached keys nobody asks for first (the cache is nearly full), the resident ones last."""
    slots = sets * ways
    chunk = max(1, min(slots + slots // 4, 1 << 18))
    rows = torch.empty(chunk, dim, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=_generator(seed))
    cold = _base(seed) + _COLD + torch.arange(slots + slots // 4, dtype=torch.int64, device="cuda")
    for k in cold.split(chunk):
        B.hps_cache_insert(h, k, rows, len(k))
    # a query between the two: with the LRU policy the cold keys are older than the resident ones
    small = [torch.zeros(1, dtype=t, device="cuda") for t in (torch.int32, torch.int64, torch.int32)]
    B.hps_cache_query(h, cold[:1], 1, rows, *small)
    for k in resident.split(chunk):
        B.hps_backing_fetch(k, len(k), dim, rows=rows)
        B.hps_cache_insert(h, k, rows, len(k))
    torch.cuda.synchronize()


def prepare(case, seed):
    s = _State(case)
    op, n, dim, sets, ways = case["op"], case["keys"], case["dim"], case["sets"], case["ways"]
    policy = case.get("policy", "counter")
    if op == "multi":
        s.handles, keys = [], []
        for t in range(case["tables"]):
            resident = _resident(sets, ways, seed * 64 + t)
            s.handles.append(s.cache(sets, ways, dim))
            _fill(s.handles[-1], sets, ways, dim, resident, seed * 64 + t)
            B.hps_cache_set_concurrent_writers(s.handles[-1], case["checked"])
            keys.append(_batches(n, resident, seed * 64 + t, 4)[0])
        s.keys = list(torch.cat(keys, dim=1).contiguous())
        s.result(case["tables"] * n, dim)
        return s
    s.h = s.cache(sets, ways, dim, policy)
    if op == "lookup":
        everything = _base(seed) + torch.arange(case["space"], dtype=torch.int64, device="cuda")
        hm = B.hps_hostmap_create(dim, 16, case["space"])
        s.closers.insert(0, lambda: B.hps_hostmap_destroy(hm))
        B.hps_hostmap_put(hm, everything.cpu().numpy(), _rows(everything, dim).cpu().numpy())
        s.fetch = B.hps_hostmap_fetch_fn()
        s.lookup = B.hps_lookup_create(s.h, n, 2.0, np.zeros(dim, np.float32), s.fetch, user=hm)
        s.closers.append(lambda lk=s.lookup: B.hps_lookup_destroy(lk))
        s.keys = list(_lookup_keys(case, seed))
        s.result(n, dim)
        for k in s.keys[-8:]:                      # a server that has been running
            B.hps_lookup(s.lookup, k, n, s.out)
        s.out.zero_()
    elif op == "stream":
        B.hps_cache_set_concurrent_writers(s.h, case["checked"])
        s.keys = list(_stream_keys(case, seed))
        s.result(n, dim)
        s.rows = torch.empty(n, dim, dtype=torch.float32, device="cuda")
        for _ in s.keys:                           # a server that has been running
            _stream_step(s)
        s.out.zero_()
    elif op == "publish":
        # twice as many keys as slots, in turns of n: what a pass inserts was evicted since its last turn
        turns = max(2, 2 * sets * ways // n)
        everything = _base(seed) + torch.arange(turns * n, dtype=torch.int64, device="cuda")
        s.keys = list(everything.view(turns, n))
        s.rows = [_publish_rows(case, seed, v) for v in (0, 1)]
        for k in s.keys[turns // 2:]:
            B.hps_cache_insert(s.h, k, s.rows[0], n)
        B.hps_cache_set_concurrent_writers(s.h, case["checked"])
        s.result(n, dim)
        # with the LRU policy what is cached so far is older than what the first pass inserts
        B.hps_cache_query(s.h, s.keys[0], 1, s.out, s.miss_idx, s.miss_keys, s.n_miss)
        s.out.zero_()
    elif op == "refresh":
        resident = _resident(sets, ways, seed)
        _fill(s.h, sets, ways, dim, resident, seed)
        B.hps_cache_set_concurrent_writers(s.h, case["checked"])
        s.dumped = torch.empty(sets * ways, dtype=torch.int64, device="cuda")
        s.n_dumped = torch.zeros(1, dtype=torch.int32, device="cuda")
        B.hps_cache_dump(s.h, 0, sets * ways, s.dumped, s.n_dumped)
        s.cached = s.dumped[:int(s.n_dumped.item())].clone()
        # the lower tiers' answer to the dump, two versions taken in turn
        s.rows = [torch.empty(len(s.cached), dim, dtype=torch.float32, device="cuda") for _ in range(2)]
        for v, r in enumerate(s.rows):
            B.hps_backing_fetch(s.cached, len(s.cached), dim, version=v + 1, rows=r)
        s.keys = list(_batches(n, resident, seed, _turns(n))[0])
        s.result(n, dim)
    else:
        resident = _resident(sets, ways, seed)
        _fill(s.h, sets, ways, dim, resident, seed)
        B.hps_cache_set_concurrent_writers(s.h, case["checked"])
        s.keys = list(_batches(n, resident, seed, _turns(n))[0])
        s.result(n, dim)
        if op == "dedup":
            s.session = B.hps_dedup_create(n)
            s.closers.append(lambda d=s.session: B.hps_dedup_destroy(d))
            s.unique = torch.zeros(n, dtype=torch.int64, device="cuda")
            s.inverse = torch.zeros(n, dtype=torch.int32, device="cuda")
            s.n_unique = torch.zeros(1, dtype=torch.int32, device="cuda")
            s.rows = torch.zeros(n, dim, dtype=torch.float32, device="cuda")
    return s


def _lookup_keys(case, seed):
    return (_base(seed) + _zipf(32 * case["keys"], case["space"], 1.2, _generator(seed))).view(32, -1)


def _stream_keys(case, seed):
    return (_base(seed) + _zipf(16 * case["keys"], _stream_space(case), 1.1, _generator(seed))).view(16, -1)


def _publish_rows(case, seed, version):
    g = _generator(2 * seed + version)
    return torch.empty(case["keys"], case["dim"], dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=g)


# ---- one pass ---------------------------------------------------------------------------------

def _stream_step(s):
    n, dim = s.case["keys"], s.case["dim"]
    B.hps_cache_query(s.h, s.next(), n, s.out, s.miss_idx, s.miss_keys, s.n_miss)
    B.hps_backing_fetch(s.miss_keys, n, dim, rows=s.rows, n_dev=s.n_miss, scatter_idx=s.miss_idx, scatter_out=s.out)
    B.hps_cache_insert_dn(s.h, s.miss_keys, s.rows, n, s.n_miss)


def run(s):
    c = s.case
    op, n = c["op"], c["keys"]
    if op == "query":
        B.hps_cache_query(s.h, s.next(), n, s.out, s.miss_idx, s.miss_keys, s.n_miss)
        return {"out": s.out, "n_miss": s.n_miss}
    if op == "multi":
        B.hps_cache_query_multi(s.handles, s.next(), n, s.out, s.miss_idx, s.miss_keys, s.n_miss)
        return {"out": s.out, "n_miss": s.n_miss}
    if op == "stream":
        _stream_step(s)
        return {"out": s.out}
    if op == "publish":
        k = s.next()
        B.hps_cache_insert(s.h, k, s.rows[0], n)
        B.hps_cache_update(s.h, k, s.rows[1], n)
        B.hps_cache_query(s.h, k, n, s.out, s.miss_idx, s.miss_keys, s.n_miss)
        return {"out": s.out, "n_miss": s.n_miss}
    if op == "refresh":
        rows = s.rows[s.turn % 2]
        B.hps_cache_dump(s.h, 0, c["sets"] * c["ways"], s.dumped, s.n_dumped)
        B.hps_cache_update(s.h, s.cached, rows, len(s.cached))
        B.hps_cache_query(s.h, s.next(), n, s.out, s.miss_idx, s.miss_keys, s.n_miss)
        return {"out": s.out, "n_miss": s.n_miss, "n_dumped": s.n_dumped}
    if op == "dedup":
        B.hps_dedup(s.session, s.next(), n, s.unique, s.inverse, s.n_unique)
        B.hps_cache_query_dn(s.h, s.unique, n, s.n_unique, s.rows, s.miss_idx, s.miss_keys, s.n_miss)
        B.hps_backing_fetch(s.miss_keys, n, c["dim"], n_dev=s.n_miss, scatter_idx=s.miss_idx, scatter_out=s.rows)
        B.hps_expand_rows(s.rows, s.inverse, n, c["dim"], s.out)
        return {"out": s.out, "n_unique": s.n_unique}
    B.hps_lookup(s.lookup, s.next(), n, s.out)
    return {"out": s.out}


# ---- what a pass cannot do without, and what it returns -----------------------------------------

def _distinct(n, space, alpha):
    """Expected number of distinct keys among n power-law draws (bins of equal width in log rank)."""
    a = 1.0 - alpha
    edge = np.unique(np.floor(np.exp(np.linspace(0.0, math.log(space + 1.0), 4096))))
    share = np.diff((edge ** a - 1.0) / (float(space + 1) ** a - 1.0))
    width = np.diff(edge)
    return float(np.sum(width * -np.expm1(n * np.log1p(-np.minimum(share / width, 1 - 1e-12)))))


def _query_bytes(n, distinct, distinct_hit, hits, ways, dim):
    return 8 * n + 8 * ways * distinct + 4 * dim * (distinct_hit + hits) + 12 * (n - hits) + 4


def work(case):
    """Bytes of one pass, each input read once and each output written once: keys, the key line of
    every distinct key, the row of every distinct cached key, the rows written, the miss list."""
    op, n, dim, sets, ways = case["op"], case["keys"], case["dim"], case["sets"], case["ways"]
    row = 4 * dim
    if op == "lookup":
        d = _distinct(n, case["space"], 1.2)
        return {"bytes": _query_bytes(n, d, d, n, ways, dim), "flops": 0}
    if op == "stream":
        # row in or out of every position; the distinct keys' rows are read (cached) or made and inserted (missing)
        d = _distinct(n, _stream_space(case), 1.1)
        return {"bytes": _query_bytes(n, d, d, n, ways, dim), "flops": 0}
    if op == "publish":
        # insert: row read and written; update: row read and written; query: row read and written
        return {"bytes": n * (3 * 8 + 3 * 8 * ways + 6 * row + 16 + 8), "flops": 0}
    hot = sets * ways / 2
    d_hit, d_miss = _distinct(HIT * n, hot, ALPHA), _distinct((1 - HIT) * n, 1 << 30, ALPHA)
    query = _query_bytes(n, d_hit + d_miss, d_hit, HIT * n, ways, dim)
    if op == "refresh":
        m = 0.87 * sets * ways                     # cached keys: key dumped and read, row read and written
        return {"bytes": sets * ways * 8 + 8 * m + m * (8 + 2 * row) + sets * (8 * ways + 8) + query, "flops": 0}
    if op == "multi":
        return {"bytes": case["tables"] * query, "flops": 0}
    if op == "dedup":
        # keys in, inverse out; the distinct rows read from the cache or made, every position's row written
        return {"bytes": 8 * n + 4 * n + (8 + 8 * ways) * (d_hit + d_miss) + row * (d_hit + n), "flops": 0}
    return {"bytes": query, "flops": 0}


def tolerance(case):
    """Rows are moved as opaque words and the stand-in's values are exact in fp32."""
    return "exact"


def exact(case, seed):
    op, n, dim, sets, ways = case["op"], case["keys"], case["dim"], case["sets"], case["ways"]

    def served(keys, hit, version=0):
        return (_rows(keys, dim, version) * hit[:, None]).double()

    if op == "multi":
        outs, misses = [], 0
        for t in range(case["tables"]):
            keys, hit = _batches(n, _resident(sets, ways, seed * 64 + t), seed * 64 + t, 4)
            outs.append(served(keys[0], hit[0]))
            misses += int((~hit[0]).sum())
        return {"out": torch.cat(outs), "n_miss": torch.tensor([misses], dtype=torch.int32)}
    if op in ("stream", "lookup"):
        keys = (_stream_keys if op == "stream" else _lookup_keys)(case, seed)
        return {"out": _rows(keys[0], dim).double()}
    if op == "publish":
        return {"out": _publish_rows(case, seed, 1).double(), "n_miss": torch.zeros(1, dtype=torch.int32)}
    keys, hit = (x[0] for x in _batches(n, _resident(sets, ways, seed), seed, _turns(n)))
    if op == "dedup":
        return {"out": _rows(keys, dim).double(), "n_unique": torch.tensor([len(torch.unique(keys))], dtype=torch.int32)}
    n_miss = torch.tensor([int((~hit).sum())], dtype=torch.int32)
    if op == "refresh":
        return {"out": served(keys, hit, version=1), "n_miss": n_miss, "n_dumped": None}
    return {"out": served(keys, hit), "n_miss": n_miss}
