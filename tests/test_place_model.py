"""The claim order of the batch inserts as a model on the CPU: threads interleave at every bucket read
and every compare-and-swap, and a read may return any state the bucket has had since the kernel
began (loads are cached).  Whatever the schedule, a key is stored once, every copy but one reports
the key as met, and nothing is lost while the table has room."""
import random

import pytest

EMPTY, TOMB = "empty", "tomb"
SLOTS = 8


class Table:
    def __init__(self, nb, rng):
        self.b = [[EMPTY] * SLOTS for _ in range(nb)]
        self.past = [[] for _ in range(nb)]     # states a stale read may return
        self.rng = rng

    def start(self):
        self.past = [[list(x)] for x in self.b]

    def read(self, i):
        return list(self.rng.choice(self.past[i]))

    def cas(self, i, c, expected, key):
        seen = self.b[i][c]
        if seen == expected:
            self.b[i][c] = key
            self.past[i].append(list(self.b[i]))
        return seen


def path(key, nb):
    home, step = hash((key, 1)) % nb, 1 + hash((key, 2)) % max(1, nb - 1)
    return [(home + s * step) % nb for s in range(nb)], (step >> 1) & 7


def pick(free, rot):
    return min(free, key=lambda c: (c - rot) % SLOTS)


def place(t, key):
    """One lane's walk: a generator that yields before every access to the table."""
    buckets, rot = path(key, len(t.b))
    at, first = 0, None
    while at < len(buckets):
        yield
        line = t.read(buckets[at])
        if key in line:
            return "met"
        e = {c for c in range(SLOTS) if line[c] == EMPTY}
        tb = {c for c in range(SLOTS) if line[c] == TOMB}
        if first is None and (e or tb):
            first = (at, e, tb)
        at += 1
        if not e and at < len(buckets):
            continue
        if first is None:
            return "full"
        at, e, tb = first
        while e or tb:                          # every slot the probe saw free, tombstones first
            c = pick(tb or e, rot)
            yield
            expected = TOMB if tb else EMPTY
            seen = t.cas(buckets[at], c, expected, key)
            if seen == expected:
                return "stored"
            if seen == key:
                return "met"
            e.discard(c)
            tb.discard(c)
        at, first = at + 1, None                # the bucket is full now
    return "full"


@pytest.mark.parametrize("nb", [1, 2, 3, 7, 11])
@pytest.mark.parametrize("seed", range(20))
def test_any_schedule_stores_each_key_once(nb, seed):
    rng = random.Random(1000 * nb + seed)
    t = Table(nb, rng)
    room = SLOTS * nb
    present = []
    for k in range(rng.randint(0, room)):       # a live and erased past, placed one key at a time
        walk = place(t, k)
        t.start()
        for _ in walk:
            pass
        present.append(k)
    for k in [k for k in present if rng.random() < 0.5]:
        for line in t.b:
            if k in line:
                line[line.index(k)] = EMPTY if EMPTY in line else TOMB
                present.remove(k)
    t.start()
    fresh = list(range(10_000, 10_000 + room - len(present)))   # at most what fits
    batch = [rng.choice(fresh + present) for _ in range(6 * room)] if fresh or present else []
    walks = [(k, place(t, k)) for k in batch]
    out = []
    while walks:
        j = rng.randrange(len(walks))
        k, w = walks[j]
        try:
            next(w)
        except StopIteration as s:
            out.append((k, s.value))
            walks.pop(j)
    stored = [x for line in t.b for x in line if x not in (EMPTY, TOMB)]
    assert len(stored) == len(set(stored))
    assert set(stored) == set(present) | set(batch)
    for k in set(batch):
        got = sorted(v for kk, v in out if kk == k)
        want = ["met"] * batch.count(k) if k in present else ["met"] * (batch.count(k) - 1) + ["stored"]
        assert got == want, (k, got)
