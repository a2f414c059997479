"""Batches whose insert and erase kernels settle the counters themselves: live count, statuses of
later copies and ranks equal the oracle's on both sides of the grid limit, below, at and beyond
capacity, with repeated and out-of-band keys."""
import numpy as np
import pytest

from test_gpu_parity import RESERVED, Pair, dev  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu


# 2049 keys are the first beyond one workgroup, 2^16 the last of 256 blocks
@pytest.mark.parametrize("n", [2049, 4097, (1 << 16) - 1, 1 << 16, (1 << 16) + 1])
@pytest.mark.parametrize("room", [-300, 0, 5000])
def test_settled_batches(dev, n, room):  # noqa: F811
    rng = rng_for(7600, n)
    keys = np.concatenate([distinct_u64(rng, n), RESERVED])
    k = keys[rng.integers(0, keys.size, size=n)]
    # the batch ends `room` slots below capacity, or meets FULL within it
    p = Pair(dev, np.unique(k).size + n // 2 + room, 64, path=ct.INSERT_RESOLVE_FIRST)
    p.insert(distinct_u64(rng_for(7601, n), n // 2), np.arange(n // 2, dtype=np.uint64))
    p.insert(k, rng.integers(0, 1 << 62, size=n, dtype=np.uint64))
    assert p.g.size() == p.o.size()
    for _ in range(2):     # the second finds nothing
        p.erase(k[::-1])
        assert p.g.size() == p.o.size()
    p.insert(k, rng.integers(0, 1 << 62, size=n, dtype=np.uint64))
    p.same_state()
