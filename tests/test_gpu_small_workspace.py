"""A workspace smaller than ct_workspace_bytes is left unused, also one that would hold another way of
running the batch: the batch runs in the table's own chunks, on the path that the table has reported."""
import ctypes as C

import numpy as np
import pytest
import torch

from test_gpu_parity import Pair, dev, g64  # noqa: F401
from test_gpu_partitioned import N, partitioned, workspace
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu


def launches(t, call):
    """Launches per kernel kind of a call."""
    t.profiling(True)
    t.profile_reset()
    assert call() == ct.CT_OK
    out = {k: n for k, (_, n) in t.profile().items()}
    t.profiling(False)
    return out


def chunks(n, chunk):
    return -(-n // chunk)


@pytest.mark.parametrize("op", ["insert", "erase"])
def test_speculative_room_after_batches_that_changed_little(dev, op):  # noqa: F811
    n = 60_000
    p = Pair(dev, 1 << 18, 64)
    k = distinct_u64(rng_for(8000), 2 * n)
    p.insert(k[:n], k[:n])
    if op == "insert":
        p.insert(k[:n], k[:n])          # all present: the next one resolves repeated keys first
    else:
        p.erase(k[n:])                  # none present: so does the next erase
    p.g.size()
    code = ct.OP_INSERT if op == "insert" else ct.OP_ERASE
    size = 13 * (1 << 16)               # what a speculative chunk of 2^16 takes
    assert workspace(p.g, code, 0, n) > size
    ws = torch.empty(size, dtype=torch.uint8, device=dev)
    part = k[2000: n + 2000] if op == "insert" else k[n - 2000: 2 * n - 2000]   # little changes again
    keys = g64(part, dev)
    flags = torch.empty(n, dtype=torch.uint8, device=dev)
    L, s = ct.lib(), ct._stream(dev)
    if op == "insert":
        got = launches(p.g, lambda: L.ct_insert_batch_ws(p.g._h, ct._ptr(keys), ct._ptr(keys), n, ct._ptr(flags),
                                                         ws.data_ptr(), size, s))
        want = p.o.insert(part, part)
    else:
        got = launches(p.g, lambda: L.ct_erase_batch_ws(p.g._h, ct._ptr(keys), n, ct._ptr(flags),
                                                        ws.data_ptr(), size, s))
        want = p.o.erase(part)
    np.testing.assert_array_equal(flags.cpu().numpy(), want)
    p.same_state()
    assert p.g.chunk == 1 << 15 and got[op] == chunks(n, p.g.chunk)
    assert got["prologue"] == got[op]   # repeated keys first


def test_room_below_that_of_a_partitioned_insert(dev):  # noqa: F811
    t = ct.Table(2 * N, ct.VAL_U64, bucket_count=N // 3, device=dev)
    assert partitioned(t, N)
    need = workspace(t, ct.OP_INSERT, 0, N)
    keys = g64(distinct_u64(rng_for(8001), N), dev)
    ws = torch.empty(need - 256, dtype=torch.uint8, device=dev)
    got = launches(t, lambda: ct.lib().ct_insert_batch_ws(t._h, ct._ptr(keys), ct._ptr(keys), N, None,
                                                          ws.data_ptr(), need - 256, ct._stream(dev)))
    assert got["insert"] == chunks(N, t.chunk) > 1
    assert t.size() == N and t.check() == 0


@pytest.mark.parametrize("op,pool", [(ct.OP_INSERT, 0), (ct.OP_ERASE, 0), (ct.OP_INSERT, 1), (ct.OP_ERASE, 1)])
def test_sizes_beyond_any_memory(dev, op, pool):  # noqa: F811
    """The largest chunk is what a batch can use, whatever its size: no power of two is looked for past
    the range of 64 bits."""
    t = ct.Table(1 << 18, ct.VAL_U32, device=dev)
    want = workspace(t, op, pool, 1 << 40)
    assert want > 0
    for n in ((1 << 62) - 1, 1 << 62, (1 << 62) + 1, (1 << 63) - 1):
        assert workspace(t, op, pool, n) == want
