"""Batches beyond the table's chunk that get no workspace: torch has no memory for it, the caller
declines it, or the batch is captured into a graph.  Same results as the oracle's in the table's own
chunks, and a request that failed is not repeated by each of the next batches."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import Pair, dev, g64, npu  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

BIG = 12 * 5000     # bytes: more than any output of the batches below, less than any workspace


@pytest.fixture
def no_memory(monkeypatch):
    """From when it is called, torch has no memory for large byte tensors; it returns the list of those
    asked for."""
    empty = torch.empty

    def start():
        asked = []

        def short(*size, **kw):
            if kw.get("dtype") is torch.uint8 and isinstance(size[0], int) and size[0] > BIG:
                asked.append(size[0])
                raise torch.cuda.OutOfMemoryError("none left")
            return empty(*size, **kw)

        monkeypatch.setattr(torch, "empty", short)
        return asked

    return start


def batches(p, rounds, seed):
    rng = rng_for(8100, seed)
    keys = distinct_u64(rng, 20_000)
    for _ in range(rounds):
        k = keys[rng.integers(0, keys.size, size=12_000)]
        p.insert(k, rng.integers(0, 1 << 62, size=k.size, dtype=np.uint64))
        p.erase(keys[rng.integers(0, keys.size, size=12_000)])
    p.same_state()


def test_no_memory_for_a_workspace(dev, no_memory, monkeypatch):  # noqa: F811
    p = Pair(dev, 30_000, 64)
    a = Pair(dev, 30_000, 32, pool=15_000)
    asked = no_memory()
    assert p.g.chunk < 12_000
    batches(p, 40, 0)
    assert 1 <= len(asked) <= 1 + 80 // 64
    keys = distinct_u64(rng_for(8101), 20_000)
    for k in (keys[:12_000], keys[6_000:18_000], np.concatenate([keys[:6_000]] * 2)):
        a.insert_alloc(k)
        a.erase_release(k[::2])
    a.same_state()
    assert len(asked) <= 3
    monkeypatch.undo()     # memory again: a workspace within the next 64 batches
    p.g._ws_rest = 1
    batches(p, 2, 1)
    assert p.g._ws_rest == 0


def test_declined_workspace(dev, no_memory):  # noqa: F811
    p = Pair(dev, 30_000, 64)
    asked = no_memory()
    p.g.workspace = False
    batches(p, 4, 2)
    assert asked == []


def test_captured_batches_beyond_the_chunk(dev):  # noqa: F811
    """Captured with no workspace, replayed with eager batches between."""
    rng = rng_for(8102)
    n = 20_000
    keys = distinct_u64(rng, 30_000)
    ins = keys[rng.integers(0, keys.size, size=n)]
    out = keys[rng.integers(0, keys.size, size=n)]
    vals = rng.integers(0, 1 << 62, size=n, dtype=np.uint64)
    t = ct.Table(40_000, ct.VAL_U64, device=dev)
    assert t.chunk < n
    gk, gv, go = g64(ins, dev), g64(vals, dev), g64(out, dev)
    t.insert(gk, gv)                       # (kernels loaded before the capture)
    t.erase(go)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        t.clear()
        st = t.insert(gk, gv)
        er = t.erase(go)
    o = oracle.OracleTable(40_000, 64, ct.HASH_MIX64, 40_000)
    want_st, want_er = o.insert(ins, vals), o.erase(out)
    ek, ev = o.dump()
    for r in range(3):
        st.fill_(7)
        er.fill_(7)
        g.replay()
        np.testing.assert_array_equal(st.cpu().numpy(), want_st)
        np.testing.assert_array_equal(er.cpu().numpy(), want_er)
        k, v = t.dump()
        order = np.argsort(npu(k), kind="stable")
        np.testing.assert_array_equal(npu(k)[order], ek)
        np.testing.assert_array_equal(npu(v)[order], ev)
        assert t.size() == o.size() and t.check() == 0
        t.insert(g64(keys[r * 500:], dev), g64(keys[r * 500:], dev))   # eager, on a workspace
        torch.cuda.synchronize()
