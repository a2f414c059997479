"""The claim order under injected losses, on the model of test_place_model.py: a key that the hook
chooses asks for the slot that it loses only after the bucket's other free slots."""
import random

import pytest

import test_place_model as model
from test_place_model import EMPTY, SLOTS, TOMB


def place(t, key):
    """place() of the model with the hook on for every second key."""
    buckets, rot = model.path(key, len(t.b))
    at, first = 0, None
    while at < len(buckets):
        yield
        line = t.read(buckets[at])
        if key in line:
            return "met"
        free = {c: line[c] for c in range(SLOTS) if line[c] in (EMPTY, TOMB)}
        if first is None and free:
            first = (at, free)
        at += 1
        if EMPTY not in free.values() and at < len(buckets):
            continue
        if first is None:
            return "full"
        at, free = first
        lose, late = key % 2 == 0, {}
        while free:
            tb = [c for c in free if free[c] == TOMB]
            c = model.pick(tb or free, rot)
            kind = free.pop(c)
            expected = kind
            if lose and c == rot:            # loses for certain: it expects the other kind of free slot
                lose, late = False, {c: kind}
                expected = TOMB if kind == EMPTY else EMPTY
            yield
            seen = t.cas(buckets[at], c, expected, key)
            if seen == expected:
                return "stored"
            if seen == key:
                return "met"
            if not free:
                free, late = late, {}
        at, first = at + 1, None
    return "full"


@pytest.mark.parametrize("nb", [1, 2, 3, 7, 11])
@pytest.mark.parametrize("seed", range(20))
def test_any_schedule_stores_each_key_once(nb, seed, monkeypatch):
    monkeypatch.setattr(model, "place", place)
    model.test_any_schedule_stores_each_key_once(nb, seed)


def test_a_chosen_key_takes_its_first_slot_last():
    for key in range(1000, 1040):
        t = model.Table(1, random.Random(key))
        rot = model.path(key, 1)[1]
        taken = []
        for n in range(SLOTS):       # the bucket fills up with other keys in the key's own order
            t.start()
            for _ in place(t, key):
                pass
            taken.append(t.b[0].index(key))
            t.b[0][taken[-1]] = ("other", n)
        order = [(rot + k) % SLOTS for k in range(SLOTS)]
        assert taken == (order[1:] + order[:1] if key % 2 == 0 else order)
