"""Large inserts of several keys per bucket bring the keys to the buckets: same results as the
oracle's with distinct, repeated, present and out-of-band keys, tombstones, bins that overflow and
a table filled to its last slot."""
import ctypes as C

import numpy as np
import pytest
import torch

from test_gpu_parity import RESERVED, Pair, dev, g64  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

N = 1 << 23   # the smallest batch that takes the path


def workspace(t, op, pool, n):
    nb = C.c_int64(0)
    assert ct.lib().ct_workspace_bytes(t._h, op, pool, n, C.byref(nb)) == ct.CT_OK
    return nb.value


def partitioned(t, n):
    """Its workspace is neither that of speculative chunks (as an erase's) nor the general one."""
    return workspace(t, ct.OP_INSERT, 0, n) not in (workspace(t, ct.OP_ERASE, 0, n),
                                                    workspace(t, ct.OP_ERASE, 1, n))


def values(rng, bits, n):
    return None if bits == 0 else rng.integers(0, 1 << 62, size=n, dtype=np.uint64).astype(
        np.uint32 if bits == 32 else np.uint64)


@pytest.mark.parametrize("kind,bits", [("full", 64), ("full", 0), ("repeated", 32), ("one_key", 64), ("one_key", 0)])
def test_partitioned_insert(dev, kind, bits):  # noqa: F811
    rng = rng_for(7400, bits + len(kind))
    n = {"full": N, "repeated": N + 77, "one_key": N + 1}[kind]
    cap = n if kind == "full" else 2 * n
    p = Pair(dev, cap, bits, path=ct.INSERT_SPECULATIVE)
    keys = np.concatenate([distinct_u64(rng, cap), RESERVED])
    if kind == "full":       # every slot ends taken: many home buckets are full
        k = keys[:n]
    else:                    # present keys and tombstones first
        p.insert(keys[:n // 2], values(rng, bits, n // 2))
        p.erase(keys[: n // 4])
        k = keys[rng.integers(0, keys.size, size=n)]
        if kind == "one_key":    # one bin overflows
            k[rng.random(n) < 0.3] = keys[0]
    assert partitioned(p.g, n)
    p.insert(k, values(rng, bits, n))
    p.same_state()
    p.find(k[::3])


def test_batches_that_stay(dev):  # noqa: F811
    """Below three keys per bucket or 2^23 keys, with a chosen chunk, beyond capacity, the spatial hash."""
    assert not partitioned(ct.Table(N, ct.VAL_U64, device=dev), N - 1)
    assert not partitioned(ct.Table(N, ct.VAL_U64, device=dev), N + 1)
    assert not partitioned(ct.Table(N, ct.VAL_U64, bucket_count=N // 3 + 1, device=dev), N)
    assert partitioned(ct.Table(N, ct.VAL_U64, bucket_count=N // 3, device=dev), N)
    assert not partitioned(ct.Table(N, ct.VAL_U64, chunk=1 << 17, device=dev), N)
    assert not partitioned(ct.Table(N, ct.VAL_U64, ct.HASH_VOXEL21, device=dev), N)


def test_partitioned_insert_without_status(dev):  # noqa: F811
    rng = rng_for(7401)
    k = g64(distinct_u64(rng, N), dev)
    t = ct.Table(2 * N, ct.VAL_U64, device=dev)
    assert partitioned(t, N)
    t.insert(k, k, status=False)
    t.insert(k[:N // 2].repeat(2), k, status=False)   # the last chunk stored every key: speculative still
    assert t.size() == N and t.check() == 0
    v, f = t.find(k)
    assert bool(f.all()) and torch.equal(v, k)
