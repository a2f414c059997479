"""Timed cases of the batch hash containers and the index pool.

Each case is work that a program using this library has it do, through the Python binding
(`paper_1908_05936_amd.ct`): lookups, updates, bulk builds, voxel frames, block allocation, a
schedule over many tables, request serving and per-thread operations.  Sizes, load factors and key
distributions are those of `workloads.py`, `bench.py` and the tests, from batches of a few keys to
the 2^26-key table.  Inputs are drawn on the GPU from a seed.

Every pass leaves its table and pool holding what they held before it (a build starts with a
clear, an update puts back what it removed, a frame's new blocks leave in reverse order), so
passes can follow one another on one state.
"""
import math
import random

import numpy as np
import torch

from paper_1908_05936_amd import ct

DEV = "cuda"
M64 = (1 << 64) - 1
LOAD = 0.8                     # live keys per slot, as the large-table workload
SLICE = 1 << 24                # elements drawn at a time: bounds the generators' temporaries
VALUE_BYTES = {"none": 0, "u32": 4, "u64": 8}
VALUE_KIND = {"none": ct.VAL_NONE, "u32": ct.VAL_U32, "u64": ct.VAL_U64}


def listed():
    return [
        # one small query batch against a small map: what a request costs before its size matters
        {"name": "find_small", "kind": "find", "entries": 1 << 16, "n": 256, "vals": "u64", "zipf": False},
        # a few hundred keys leave a map and come back: latency of the updating calls
        {"name": "update_small", "kind": "churn", "entries": 1 << 16, "n": 500, "vals": "u32"},
        # the plain-table workload: build 2^16 keys, find, erase a quarter, find again
        {"name": "plain_table", "kind": "plain", "entries": 1 << 16, "vals": "u32"},
        # the large-table lookup: Zipf popularity, a fifth of the keys absent
        {"name": "find_zipf_large", "kind": "find", "entries": 1 << 26, "n": 1 << 27, "vals": "u64", "zipf": True},
        # an unordered_set collects the distinct keys of a batch that repeats each about four times
        {"name": "set_repeated", "kind": "fill", "entries": 1000003, "repeat": 4, "vals": "none"},
        # the large-table build: clear, then 2^26 distinct keys in one call to load factor 0.8
        {"name": "fill_large", "kind": "fill", "entries": 1 << 26, "repeat": 1, "vals": "u64"},
        # the large-table churn: 2^24 keys erased and inserted again at load factor 0.8
        {"name": "churn_large", "kind": "churn", "entries": 1 << 26, "n": 1 << 24, "vals": "u64"},
        # a reconstruction frame: find 2^18 blocks, allocate the missing tenth, release what leaves
        {"name": "voxel_frame", "kind": "frame", "resident": 1 << 20, "n": 1 << 18, "miss": 0.1},
        # block allocation from raw surface samples: several samples fall into each new block
        {"name": "blocks_alloc", "kind": "blocks", "resident": 1 << 20, "n": 1 << 21, "repeat": 4},
        # the multi-table schedule, grouped, with the tuned settings (merged runs, one chunk per batch)
        {"name": "multi_table", "kind": "multi", "tables": 256, "entries_hi": 20, "batch_hi": 18, "sizes": 4},
        # requests of uneven size for many tables, from host memory through the request server
        {"name": "serve_requests", "kind": "serve", "tables": 16, "requests": 96, "req_hi": 18, "sizes": 5},
        # per-thread operations inside kernels: insert, find and erase through the device functions
        {"name": "device_ops", "kind": "device", "entries": 1 << 23, "vals": "u64"},
    ]


def draw(rng: random.Random):
    def size(lo, hi):
        return max(1, int(round(2.0 ** rng.uniform(lo, hi))))

    kind = rng.choice(["find", "find", "churn", "churn", "plain", "fill", "fill", "frame", "blocks", "multi",
                       "serve", "device"])
    vals = rng.choice(["none", "u32", "u64"])
    if kind == "find":
        return {"kind": kind, "entries": size(10, 26), "n": size(4, 26), "vals": vals, "zipf": rng.random() < 0.5}
    if kind == "churn":
        entries = size(10, 26)
        return {"kind": kind, "entries": entries, "n": min(size(4, 24), max(1, entries // 4)), "vals": vals}
    if kind == "plain":
        return {"kind": kind, "entries": size(10, 20), "vals": vals}
    if kind == "fill":
        repeat = rng.choice([1, 1, 2, 4])
        return {"kind": kind, "entries": size(10, 26 - math.log2(repeat)), "repeat": repeat, "vals": vals}
    if kind == "frame":
        resident = size(14, 21)
        return {"kind": kind, "resident": resident, "n": min(size(10, 19), resident // 2),
                "miss": rng.choice([0.02, 0.1, 0.3])}
    if kind == "blocks":
        return {"kind": kind, "resident": size(12, 21), "n": size(8, 22), "repeat": rng.choice([1, 2, 4, 8])}
    if kind == "multi":
        return {"kind": kind, "tables": rng.randint(16, 256), "entries_hi": rng.randint(14, 20),
                "batch_hi": rng.randint(12, 18), "sizes": rng.randint(0, 999)}
    if kind == "serve":
        return {"kind": kind, "tables": rng.randint(4, 16), "requests": rng.randint(16, 96),
                "req_hi": rng.randint(12, 18), "sizes": rng.randint(0, 999)}
    return {"kind": kind, "entries": size(12, 23), "vals": vals}


# --- inputs ---------------------------------------------------------------------------------------
def _gen(seed, stream=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + stream)
    return g


def _i64(x):
    """A 64-bit pattern as the Python int torch.int64 holds it as."""
    x &= M64
    return x - (1 << 64) if x >> 63 else x


def _shr(z, s):
    return (z >> s) & ((1 << (64 - s)) - 1)


def _key(seed, idx):
    """Key number idx of a seed: splitmix64 outputs, so distinct numbers are distinct keys.  `seed`
    is an int or an int64 tensor, one per element."""
    z = (idx + 1) * _i64(0x9E3779B97F4A7C15)
    z += _i64(seed * 0x632BE59BD9B4E019) if isinstance(seed, int) else seed * _i64(0x632BE59BD9B4E019)
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _uniform(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _ranks(u, n, s=1.1):
    """Zipf(s) ranks in [0, n) by the continuous inverse of the popularity."""
    a = 1.0 - s
    lo, hi = 0.5 ** a, (n + 0.5) ** a
    return ((lo + u * (hi - lo)) ** (1.0 / a) + 0.5).long().clamp_(1, n) - 1


def _scatter(rank, n, seed):
    """Popularity rank -> key number, a permutation of [0, n)."""
    a = (0x9E3779B1 + 2 * seed) % n | 1
    while math.gcd(a, n) != 1:
        a += 2
    return (rank * a + seed) % n


def _queries(seed, entries, n, zipf, absent=0.2):
    """Key numbers of n queries: below `entries` present, at or above it absent."""
    out = torch.empty(n, dtype=torch.int64, device=DEV)
    g = _gen(seed, 1)
    for c in range(0, n, SLICE):
        m = min(SLICE, n - c)
        u = _uniform(g, m)
        j = _scatter(_ranks(u, entries), entries, seed) if zipf else (u * entries).long()
        fresh = entries + torch.arange(c, c + m, device=DEV)
        out[c:c + m] = torch.where(_uniform(g, m) < absent, fresh, j)
    return out


def _keys(seed, idx):
    out = torch.empty_like(idx)
    for c in range(0, idx.numel(), SLICE):
        out[c:c + SLICE] = _key(seed, idx[c:c + SLICE])
    return out


def _vals(idx, vals, salt=0):
    """Values of the given key numbers in the width of the map (None for a set)."""
    if vals == "none":
        return None
    v = idx + (salt << 20)
    return v.to(torch.int32) if vals == "u32" else v


def _expect(idx, hit, vals, salt=0):
    """What a find of these key numbers returns (sentinel: all ones)."""
    if vals == "none":
        return None
    v = _vals(idx, vals, salt)
    return torch.where(hit, v, torch.full_like(v, -1))


def _capacity(entries):
    return max(1, int(round(entries / LOAD)))


def _filled(seed, entries, vals):
    t = ct.Table(_capacity(entries), VALUE_KIND[vals], ct.HASH_MIX64, device=DEV)
    idx = torch.arange(entries, device=DEV)
    t.insert(_keys(seed, idx), _vals(idx, vals), status=False)
    return t


def _read_back(seed, idx, entries):
    """Key numbers looked up after an update: about one in sixteen of the updated, half of those
    replaced by numbers that are not there."""
    s = idx[::16]
    fresh = entries + torch.arange(s.numel(), device=DEV)
    return torch.where(_uniform(_gen(seed, 9), s.numel()) < 0.5, s, fresh)


def _surface(p, width, seed):
    """Packed block coordinates of surface block number p: a height field over a strip `width`
    blocks wide that the camera moves along, so consecutive numbers are neighbours and distinct
    numbers distinct blocks."""
    x = p // width
    y = p % width
    z = (60.0 * torch.sin(x.double() / 37.0 + seed) + 45.0 * torch.cos(y.double() / 29.0)).floor().long()
    m = (1 << 21) - 1
    return ((x - 1024) & m) | (((y - width // 2) & m) << 21) | ((z & m) << 42)


def _first(idx):
    """For each element whether it is the first with its number, and the number's rank in that order."""
    _, inv = torch.unique(idx, return_inverse=True)
    n = idx.numel()
    pos = torch.arange(n, device=idx.device)
    low = torch.full((int(inv.max()) + 1,), n, dtype=torch.int64, device=idx.device)
    low.scatter_reduce_(0, inv, pos, "amin")
    first = low[inv] == pos
    order = torch.cumsum(first.long(), 0) - 1
    return first, order[low[inv]], low[inv]


def _fill_idx(case, seed):
    n = case["entries"] * case["repeat"]
    if case["repeat"] == 1:
        return torch.arange(n, device=DEV)
    return (_uniform(_gen(seed, 2), n) * case["entries"]).long()


def _plain_inputs(case, seed):
    e = case["entries"]
    g = _gen(seed, 3)
    q1 = _queries(seed, e, e, False, 0.5)
    gone = torch.randperm(e, generator=g, device=DEV)[: e // 4]
    q2 = torch.randperm(e, generator=g, device=DEV)
    return q1, gone, q2


def _churn_idx(case, seed):
    g = _gen(seed, 4)
    e, n = case["entries"], case["n"]
    if n * 64 > e:
        return torch.randperm(e, generator=g, device=DEV)[:n].clone()
    start = int(torch.randint(0, e, (1,), generator=g, device=DEV))
    return (start + torch.arange(n, device=DEV) * (e // n)) % e


def _frame_idx(case, seed):
    """Block numbers a frame asks for: the trailing window of the residents, then the next unseen."""
    g = _gen(seed, 5)
    r, n = case["resident"], case["n"]
    misses = max(1, int(round(n * case["miss"])))
    hits = min(n - misses, r // 2)
    old = r - 1 - torch.randperm(r // 2, generator=g, device=DEV)[:hits]
    new = r + torch.arange(misses, device=DEV)
    q = torch.cat([old, new])
    return q[torch.randperm(q.numel(), generator=g, device=DEV)]


def _blocks_idx(case, seed):
    """Block number of each surface sample: samples wander forward over `n / repeat` new blocks,
    each of which is met at least once."""
    g = _gen(seed, 6)
    n, span = case["n"], max(1, case["n"] // case["repeat"])
    again = (_uniform(g, n - span) * span).long()
    b = torch.cat([torch.arange(span, device=DEV), again])
    return case["resident"] + b[torch.argsort(b + _uniform(g, n) * (0.1 * span))]


def _block_map(seed, resident, new):
    """A block map with room for both, its residents allocated from the pool."""
    room = 1 << max(10, math.ceil(math.log2(resident + new)))
    pool = ct.Pool(room, device=DEV)
    t = ct.Table(room, ct.VAL_U32, ct.HASH_VOXEL21, bucket_count=max(room // 2, 128), device=DEV)
    width = max(64, int(math.sqrt(resident)))
    t.insert_alloc(pool, _surface(torch.arange(resident, device=DEV), width, seed % 7))
    return t, pool, width


class _Schedule:
    """Operations over many tables, as the multi-table and serving workloads draw them: key numbers
    of all operations in one array.  The case fixes the sizes, the seed the keys."""

    def __init__(self, seed, entries, ops):
        self.entries, self.ops = entries, ops               # ops: (table, kind, n)
        self.start = np.cumsum([0] + [-(-o[2] // 16) * 16 for o in ops])  # arrays start on 16 elements
        self.total = int(self.start[-1])
        self.seed = seed

    def numbers(self, zipf):
        """(key number, table) per element.  Fills take each number once; finds and inserts ask half
        for live and half for fresh numbers, erases for live ones.  `zipf`: every operation draws
        from twice the entries by popularity."""
        g = _gen(self.seed, 7)
        lens = torch.tensor(np.diff(self.start), device=DEV)
        rep = lambda v: torch.repeat_interleave(torch.tensor(v, device=DEV), lens)  # noqa: E731
        table = rep([o[0] for o in self.ops])
        e = rep([self.entries[o[0]] for o in self.ops])
        at = torch.arange(self.total, device=DEV)
        u = _uniform(g, self.total)
        if zipf:
            return (_ranks(u, 1 << 24) * 0x9E3779B1 + table) % (2 * e), table
        kind = rep([["fill", "find", "insert", "erase"].index(o[1]) for o in self.ops])
        pos = [o[3] if o[1] == "fill" else 0 for o in self.ops]
        first = at - rep(self.start[:-1].tolist()) + rep(pos)
        fresh = (kind != 3) & (_uniform(g, self.total) < 0.5)
        live = (u * e).long()
        return torch.where(kind == 0, first, torch.where(fresh, e + at, live)), table


def _multi_schedule(case, seed):
    r = np.random.Generator(np.random.PCG64(case["sizes"]))
    logu = lambda lo, hi: int(round(2.0 ** r.uniform(lo, hi)))  # noqa: E731
    entries, loads, per = [], [], []
    for t in range(case["tables"]):
        e = logu(10, case["entries_hi"])
        ops, pos = [], 0
        while pos < e:
            b = min(logu(6, case["batch_hi"]), e - pos)
            ops.append((t, "fill", b, pos))
            pos += b
        for _ in range(4):
            ops.append((t, str(r.choice(["insert", "find", "erase"], p=[0.2, 0.7, 0.1])),
                        logu(6, case["batch_hi"]), 0))
        entries.append(e)
        loads.append(float(r.uniform(0.5, 0.9)))
        per.append(ops)
    order = np.concatenate([np.full(len(o), t) for t, o in enumerate(per)])
    r.shuffle(order)
    nxt, ops = [0] * len(per), []
    for t in order:
        ops.append(per[t][nxt[t]])
        nxt[t] += 1
    return _Schedule(seed, entries, ops), loads


def _serve_schedule(case, seed):
    r = np.random.Generator(np.random.PCG64(case["sizes"]))
    entries = [int(round(2.0 ** r.uniform(14, 22))) for _ in range(case["tables"])]
    ops = [(int(r.integers(case["tables"])), str(r.choice(["insert", "find", "erase"], p=[0.2, 0.7, 0.1])),
            int(round(2.0 ** r.uniform(8, case["req_hi"]))), 0) for _ in range(case["requests"])]
    return _Schedule(seed, entries, ops)


# --- what a program has in hand before the call ---------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "find":
        idx = _queries(seed, case["entries"], case["n"], case["zipf"])
        return {"kind": kind, "t": _filled(seed, case["entries"], case["vals"]), "q": _keys(seed, idx)}
    if kind == "churn":
        idx = _churn_idx(case, seed)
        return {"kind": kind, "t": _filled(seed, case["entries"], case["vals"]), "k": _keys(seed, idx),
                "v": _vals(idx, case["vals"], seed % 64), "q": _keys(seed, _read_back(seed, idx, case["entries"]))}
    if kind == "plain":
        e = case["entries"]
        q1, gone, q2 = _plain_inputs(case, seed)
        idx = torch.arange(e, device=DEV)
        return {"kind": kind, "t": ct.Table(2 * e, VALUE_KIND[case["vals"]], device=DEV), "k": _keys(seed, idx),
                "v": _vals(idx, case["vals"]), "q1": _keys(seed, q1), "gone": _keys(seed, gone),
                "q2": _keys(seed, q2)}
    if kind == "fill":
        idx = _fill_idx(case, seed)
        at = torch.arange(idx.numel(), device=DEV)
        k = _keys(seed, idx)
        return {"kind": kind, "t": ct.Table(_capacity(case["entries"]), VALUE_KIND[case["vals"]], device=DEV),
                "k": k, "v": _vals(at, case["vals"], seed % 64),
                "q": _keys(seed, _read_back(seed, idx, case["entries"]))}
    if kind == "frame":
        q = _frame_idx(case, seed)
        t, pool, width = _block_map(seed, case["resident"], case["n"])
        leave = q[q >= case["resident"]].flip(0)
        n = q.numel()
        return {"kind": kind, "t": t, "pool": pool, "q": _surface(q, width, seed % 7),
                "leave": _surface(leave, width, seed % 7),
                "out": torch.full((n,), -1, dtype=torch.int32, device=DEV),
                "st": torch.full((n,), 255, dtype=torch.uint8, device=DEV)}
    if kind == "blocks":
        idx = _blocks_idx(case, seed)
        t, pool, width = _block_map(seed, case["resident"], case["n"])
        first = _first(idx)[0]
        return {"kind": kind, "t": t, "pool": pool, "k": _surface(idx, width, seed % 7),
                "leave": _surface(idx[first].flip(0), width, seed % 7)}
    if kind == "multi":
        return _prepare_multi(case, seed)
    if kind == "serve":
        return _prepare_serve(case, seed)
    e = case["entries"]
    idx = torch.arange(e, device=DEV)
    q = _queries(seed, e, e, False)
    return {"kind": "device", "t": ct.Table(_capacity(e), VALUE_KIND[case["vals"]], device=DEV),
            "k": _keys(seed, idx), "v": _vals(idx, case["vals"]), "q": _keys(seed, q),
            "gone": _keys(seed, torch.randperm(e, generator=_gen(seed, 8), device=DEV)[: e // 4])}


def _prepare_multi(case, seed):
    sch, loads = _multi_schedule(case, seed)
    number, table = sch.numbers(zipf=False)
    keys = _key(table * 1000003 + seed, number)
    vals = (number * 7 + 3).to(torch.int32)
    flags = torch.zeros(sch.total, dtype=torch.uint8, device=DEV)
    vout = torch.zeros(sch.total, dtype=torch.int32, device=DEV)
    biggest = [1] * case["tables"]
    for t, _, n, _ in sch.ops:
        biggest[t] = max(biggest[t], n)
    tables = []
    for e, load, b in zip(sch.entries, loads, biggest):
        cap = math.ceil(e / load)
        tables.append(ct.Table(cap, ct.VAL_U32, ct.HASH_MIX64, bucket_count=math.ceil(cap * 1.5 / 8),
                               chunk=max(1024, 1 << math.ceil(math.log2(b))), device=DEV))
    plan = ct.Plan(device=DEV)
    for t in tables:
        plan.add(t, ct.OP_CLEAR)
    op = {"fill": ct.OP_INSERT, "insert": ct.OP_INSERT, "find": ct.OP_FIND, "erase": ct.OP_ERASE}
    for (t, kind, n, _), s in zip(sch.ops, sch.start):
        part = slice(int(s), int(s) + n)
        plan.add(tables[t], op[kind], keys=keys[part], vals=vals[part] if op[kind] == ct.OP_INSERT else None,
                 vals_out=vout[part] if kind == "find" else None, flags_out=flags[part])
    plan.group(merge_runs=True)
    return {"kind": "multi", "plan": plan, "flags": flags, "vout": vout}


def _prepare_serve(case, seed):
    sch = _serve_schedule(case, seed)
    number, table = sch.numbers(zipf=True)
    keys = _key(table * 1000003 + seed, number).cpu().pin_memory()
    vals = torch.arange(sch.total, dtype=torch.int64).pin_memory()
    flags = torch.zeros(sch.total, dtype=torch.uint8, pin_memory=True)
    vout = torch.zeros(sch.total, dtype=torch.int64, pin_memory=True)
    tables = []
    for t, e in enumerate(sch.entries):     # the first half of each table's numbers is resident
        tables.append(ct.Table(4 * e, ct.VAL_U64, device=DEV))
        idx = torch.arange(e, device=DEV)
        tables[-1].insert(_key(t * 1000003 + seed, idx), idx, status=False)
    torch.cuda.synchronize()
    server = ct.NativeServer(tables, 1 << 28, device=DEV)
    op = {"insert": ct.OP_INSERT, "find": ct.OP_FIND, "erase": ct.OP_ERASE}
    reqs = []
    for (t, kind, n, _), s in zip(sch.ops, sch.start):
        part = slice(int(s), int(s) + n)
        reqs.append((t, op[kind], keys[part], vals[part] if kind == "insert" else None,
                     vout[part] if kind == "find" else None, flags[part]))
    return {"kind": "serve", "server": server, "reqs": reqs, "flags": flags, "vout": vout}


# --- one pass -------------------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind == "find":
        v, f = state["t"].find(state["q"])
        return {"values": v, "found": f}
    if kind == "churn":
        t = state["t"]
        erased = t.erase(state["k"])
        status = t.insert(state["k"], state["v"])
        v, f = t.find(state["q"])
        return {"erased": erased, "status": status, "values": v, "found": f}
    if kind == "plain":
        t = state["t"]
        t.clear()
        status = t.insert(state["k"], state["v"])
        v1, f1 = t.find(state["q1"])
        erased = t.erase(state["gone"])
        v2, f2 = t.find(state["q2"])
        return {"status": status, "v1": v1, "f1": f1, "erased": erased, "v2": v2, "f2": f2}
    if kind == "fill":
        t = state["t"]
        t.clear()
        status = t.insert(state["k"], state["v"])
        v, f = t.find(state["q"])
        return {"status": status, "values": v, "found": f}
    if kind == "frame":
        t, pool = state["t"], state["pool"]
        v, f = t.find(state["q"])
        out, st = t.insert_alloc_masked(pool, state["q"], f, out=state["out"], status=state["st"])
        return {"values": v, "found": f, "new": out, "status": st, "released": t.erase_release(pool, state["leave"])}
    if kind == "blocks":
        t, pool = state["t"], state["pool"]
        out, st = t.insert_alloc(pool, state["k"])
        return {"values": out, "status": st, "released": t.erase_release(pool, state["leave"])}
    if kind == "multi":
        state["plan"].launch_grouped()
        return {"flags": state["flags"], "values": state["vout"]}
    if kind == "serve":
        server = state["server"]
        for r in state["reqs"]:
            server.submit(*r)
        server.wait_idle()
        server.poll()
        return {"flags": state["flags"], "values": state["vout"]}
    t = state["t"]
    t.clear()
    inserted, _ = t.dev_apply(ct.OP_INSERT, state["k"], state["v"])
    found, v = t.dev_apply(ct.OP_FIND, state["q"])
    erased, _ = t.dev_apply(ct.OP_ERASE, state["gone"])
    return {"inserted": inserted, "values": v, "found": found, "erased": erased}


# --- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    """Bytes: every input array read once, every output array written once, and the 128-byte table
    lines that the keys fall into, each at most once per operation and direction."""
    kind = case["kind"]
    vb = VALUE_BYTES[case.get("vals", "u32")]

    def lines(n, slots):
        nb = max(1.0, slots / 8.0)
        return 128.0 * nb * -math.expm1(-n / nb)      # expected lines that n random keys touch

    if kind == "find":
        n, slots = case["n"], _capacity(case["entries"])
        return {"bytes": n * (9.0 + vb) + lines(n, slots), "flops": 0.0}
    if kind == "churn":
        n, slots = case["n"], _capacity(case["entries"])
        return {"bytes": n * (9.0 + 9.0 + vb) + 4 * lines(n, slots) + n / 16 * (9.0 + vb), "flops": 0.0}
    if kind == "plain":
        e = case["entries"]
        b = 16.0 * 2 * e + e * (9.0 + vb) + 2 * lines(e, 2 * e)          # clear and build
        b += 2 * (e * (9.0 + vb) + lines(e, 2 * e)) + e / 4 * 9.0 + 2 * lines(e / 4, 2 * e)
        return {"bytes": b, "flops": 0.0}
    if kind == "fill":
        e, n = case["entries"], case["entries"] * case["repeat"]
        slots = _capacity(e)
        return {"bytes": 16.0 * slots + n * (9.0 + vb) + lines(n, slots) + n / 16 * (9.0 + vb), "flops": 0.0}
    if kind == "frame":
        n, room = case["n"], 4.0 * (1 << max(10, math.ceil(math.log2(case["resident"] + case["n"]))))
        m = max(1, int(round(n * case["miss"])))
        return {"bytes": n * (9.0 + 4) + lines(n, room) + n * 9.0 + m * (5.0 + 9.0 + 8.0) + 3 * lines(m, room),
                "flops": 0.0}
    if kind == "blocks":
        n, m = case["n"], max(1, case["n"] // case["repeat"])
        room = 4.0 * (1 << max(10, math.ceil(math.log2(case["resident"] + n))))
        return {"bytes": n * (9.0 + 4) + m * (9.0 + 8.0) + 4 * lines(m, room), "flops": 0.0}
    if kind in ("multi", "serve"):
        sch = _multi_schedule(case, 1)[0] if kind == "multi" else _serve_schedule(case, 1)
        wide = 4 if kind == "multi" else 8
        b = sum(o[2] * (9.0 + (wide if o[1] != "erase" else 0)) +
                (1 if o[1] == "find" else 2) * lines(o[2], 2.0 * sch.entries[o[0]]) for o in sch.ops)
        return {"bytes": float(b), "flops": 0.0}
    e = case["entries"]
    slots = _capacity(e)
    b = 16.0 * slots + e * (9.0 + vb) + 2 * lines(e, slots) + e * (9.0 + vb) + lines(e, slots)
    return {"bytes": b + e / 4 * 9.0 + 2 * lines(e / 4, slots), "flops": 0.0}


# --- the same results without the library ---------------------------------------------------------
def _u8(x):
    return x.to(torch.uint8)


def exact(case, seed):
    kind, vals = case["kind"], case.get("vals", "u32")
    if kind == "find":
        idx = _queries(seed, case["entries"], case["n"], case["zipf"])
        hit = idx < case["entries"]
        return {"values": _expect(idx, hit, vals), "found": _u8(hit)}
    if kind == "churn":
        idx = _churn_idx(case, seed)
        ones = torch.ones(idx.numel(), dtype=torch.uint8, device=DEV)
        q = _read_back(seed, idx, case["entries"])
        hit = q < case["entries"]
        return {"erased": ones, "status": ones, "values": _expect(q, hit, vals, seed % 64), "found": _u8(hit)}
    if kind == "plain":
        e = case["entries"]
        q1, gone, q2 = _plain_inputs(case, seed)
        dead = torch.zeros(e, dtype=torch.bool, device=DEV)
        dead[gone] = True
        h1, h2 = q1 < e, ~dead[q2]
        return {"status": torch.ones(e, dtype=torch.uint8, device=DEV), "v1": _expect(q1, h1, vals), "f1": _u8(h1),
                "erased": torch.ones(gone.numel(), dtype=torch.uint8, device=DEV),
                "v2": _expect(q2, h2, vals), "f2": _u8(h2)}
    if kind == "fill":
        idx = _fill_idx(case, seed)
        n = idx.numel()
        if case["repeat"] == 1:
            first, low = torch.ones(n, dtype=torch.bool, device=DEV), torch.arange(n, device=DEV)
        else:
            first, _, low = _first(idx)
        hit = _read_back(seed, idx, case["entries"]) < case["entries"]
        return {"status": _u8(first), "values": _expect(low[::16], hit, vals, seed % 64), "found": _u8(hit)}
    if kind == "frame":
        q, r = _frame_idx(case, seed), case["resident"]
        hit = q < r
        rank = torch.cumsum((~hit).long(), 0) - 1
        n = q.numel()
        new = torch.where(hit, torch.full_like(q, -1), r + rank).to(torch.int32)
        return {"values": _expect(q, hit, "u32"), "found": _u8(hit), "new": new,
                "status": torch.where(hit, torch.full((n,), 255, device=DEV), torch.ones(n, device=DEV)).to(torch.uint8),
                "released": torch.ones(int((~hit).sum()), dtype=torch.uint8, device=DEV)}
    if kind == "blocks":
        first, order, _ = _first(_blocks_idx(case, seed))
        return {"values": (case["resident"] + order).to(torch.int32), "status": _u8(first),
                "released": torch.ones(int(first.sum()), dtype=torch.uint8, device=DEV)}
    if kind in ("multi", "serve"):
        return None        # replaying every operation one key at a time takes minutes
    e = case["entries"]
    q = _queries(seed, e, e, False)
    hit = q < e
    return {"inserted": torch.ones(e, dtype=torch.uint8, device=DEV), "values": _expect(q, hit, vals),
            "found": _u8(hit), "erased": torch.ones(e // 4, dtype=torch.uint8, device=DEV)}
