"""Batches enqueued ahead of the device, around a full table: whichever way the host or the device
picks for a chunk, every status stays exact."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import dev, g64  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,n", [(3000, 700), (5000, 2500), (200, 199)])
def test_unsynchronised_churn_at_capacity(dev, cap, n):  # noqa: F811
    """100 rounds of inserts and erases enqueued back to back around a full table: every status
    equals the oracle's, and no internal check fails."""
    rng = rng_for(7400, cap)
    t = ct.Table(cap, ct.VAL_U64, device=dev)
    o = oracle.OracleTable(cap, 64)
    keys = distinct_u64(rng, cap + cap // 2)
    keys[:2] = [(1 << 64) - 1, (1 << 64) - 2]       # the out-of-band keys come and go too
    got, want = [], []
    for r in range(100):
        k = keys[rng.integers(0, keys.size, size=n)]
        v = rng.integers(0, 1 << 62, size=n, dtype=np.uint64)
        got.append(t.insert(g64(k, dev), g64(v, dev)))
        want.append(o.insert(k, v))
        e = keys[rng.integers(0, keys.size, size=n if r % 3 else n // 4)]
        got.append(t.erase(g64(e, dev)))
        want.append(o.erase(e))
        if r % 64 == 63:
            torch.cuda.synchronize()
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a.cpu().numpy(), b)
    assert t.size() == o.size() and t.check() == 0
    assert not t.error() & 0x80000000


@pytest.mark.parametrize("path", [ct.INSERT_AUTO, ct.INSERT_SPECULATIVE, ct.INSERT_RESOLVE_FIRST])
def test_large_chunks_decided_on_the_device(dev, path):  # noqa: F811
    """Chunks of 2^22 keys that the host cannot bound: new keys (the speculative way), a chunk with
    repeats that ends at capacity, then FULL; the out-of-band keys among them."""
    n = 1 << 22
    cap = n + 1000
    rng = rng_for(7403)
    t = ct.Table(cap, ct.VAL_U32, chunk=n, device=dev)
    t.set_insert_path(path)
    o = oracle.OracleTable(cap, 32)
    keys = distinct_u64(rng, n + 3000)
    keys[5:7] = [(1 << 64) - 1, (1 << 64) - 2]
    rep = keys[rng.integers(0, keys.size, size=n)]          # repeats, some beyond capacity

    def both(k, what):
        if what == "insert":
            v = np.arange(k.size, dtype=np.uint32)
            vt = torch.from_numpy(v.view(np.int32)).to(dev)
            return t.insert(g64(k, dev), vt), o.insert(k, v)
        return t.erase(g64(k, dev)), o.erase(k)

    # no host reads between the batches: the host's bound passes the capacity with the second insert
    out = [both(keys[:n], "insert"), both(keys[: n // 2], "erase"), both(keys[: n // 4], "insert"),
           both(rep, "insert"), both(keys[n - 5:], "insert"), both(rep, "erase"), both(keys[:n], "insert")]
    for a, b in out:
        np.testing.assert_array_equal(a.cpu().numpy(), b)
    assert t.size() == o.size() and t.check() == 0
    assert not t.error() & 0x80000000
