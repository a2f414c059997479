"""Batches larger than a default table's chunk run on a workspace in larger chunks: same results as
the oracle's at the sizes where the chunk changes, with repeated keys and beyond capacity."""
import ctypes as C

import numpy as np
import pytest
import torch

from test_gpu_parity import RESERVED, Pair, dev, g64  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

# a table of 5000 has chunks of 1024; 2^16 is where chunks resolve repeated keys through bins
SIZES = [1024, 1025, 4097, (1 << 16) - 1, (1 << 16) + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("cap", [5000, 60_000])
def test_batches_beyond_the_chunk(dev, cap, n):  # noqa: F811
    rng = rng_for(7300, n)
    p = Pair(dev, cap, 32, pool=cap // 2)
    keys = np.concatenate([distinct_u64(rng, max(cap // 2, 2000)), RESERVED])
    p.insert_alloc(keys[rng.integers(0, keys.size, size=n)])
    p.erase_release(keys[rng.integers(0, keys.size, size=n)])
    p.same_state()
    q = Pair(dev, cap, 64)
    for _ in range(2):
        k = keys[rng.integers(0, keys.size, size=n)]
        q.insert(k, rng.integers(0, 1 << 62, size=n, dtype=np.uint64))
        q.erase(keys[rng.integers(0, keys.size, size=n)])
    q.same_state()


def test_batch_beyond_the_workspace_chunk(dev):  # noqa: F811
    """2^21 keys is the largest workspace chunk: a batch just beyond it takes two."""
    rng = rng_for(7301)
    n = (1 << 21) + 77
    p = Pair(dev, 1 << 20, 32)
    keys = distinct_u64(rng, (1 << 20) + 500)   # the last 500 meet a full table
    k = keys[rng.integers(0, keys.size, size=n)]
    p.insert(k, np.arange(n, dtype=np.uint32))
    p.erase(k[: n // 2][::-1])
    p.same_state()


def test_speculative_batch_beyond_its_chunk(dev):  # noqa: F811
    """2^23 keys is the largest speculative chunk: copies of a key on both sides of its end."""
    rng = rng_for(7303)
    n = (1 << 23) + 77
    p = Pair(dev, n + 1000, 32, bucket_count=n // 2, path=ct.INSERT_SPECULATIVE)
    keys = np.concatenate([distinct_u64(rng, n - 2), RESERVED])
    k = keys[rng.permutation(n)]
    k[-70:] = k[:70]
    p.insert(k, np.arange(n, dtype=np.uint32))
    p.erase(k[::-1])
    p.same_state()


def test_workspace_arguments(dev):  # noqa: F811
    t = ct.Table(5000, ct.VAL_NONE, device=dev)
    nb = C.c_int64(0)
    L = ct.lib()
    assert L.ct_workspace_bytes(t._h, ct.OP_INSERT, 0, t.chunk, C.byref(nb)) == ct.CT_OK and nb.value == 0
    assert L.ct_workspace_bytes(t._h, ct.OP_INSERT, 0, t.chunk + 1, C.byref(nb)) == ct.CT_OK and nb.value > 0
    assert L.ct_workspace_bytes(t._h, ct.OP_INSERT, 0, -1, C.byref(nb)) == ct.CT_E_INVALID
    keys = g64(distinct_u64(rng_for(7302), 3000), dev)
    ws = torch.empty(nb.value, dtype=torch.uint8, device=dev)
    args = (t._h, ct._ptr(keys), None, 3000, None)
    s = ct._stream(dev)
    assert L.ct_insert_batch_ws(*args, ws.data_ptr() + 8, nb.value - 8, s) == ct.CT_E_INVALID
    assert L.ct_insert_batch_ws(*args, ws.data_ptr(), 256, s) == ct.CT_OK       # too small: unused
    assert t.size() == 3000 and t.check() == 0
    own = ct.Table(5000, ct.VAL_NONE, chunk=1024, device=dev)                   # a chosen chunk stays
    assert L.ct_workspace_bytes(own._h, ct.OP_INSERT, 0, 4096, C.byref(nb)) == ct.CT_OK and nb.value == 0
