"""The wave-cooperative probe round at the sizes where it can go wrong: batches around the lanes of
a wave (64), of a packed round (32, 16, 8) and of a group, on tables of one bucket and up, in every
probe-step mode, with full buckets and tombstones.  Against the oracle, bit exact."""
import numpy as np
import pytest

from test_gpu_parity import RESERVED, Pair, dev  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 255, 256, 257, 1000,
         1023, 1025, 2047, 2048, 2049]   # up to 2048 updates run as one workgroup
# (capacity, buckets): one bucket, a power of two, a prime, neither (linear steps); all physically
# full or nearly, so that absent keys walk several buckets
TABLES = [(8, 1), (64, 8), (104, 13), (72, 9), (1000, 0)]


@pytest.mark.parametrize("bits", [0, 32, 64])
@pytest.mark.parametrize("cap,nb", TABLES)
def test_find_batch_sizes(dev, cap, nb, bits):  # noqa: F811
    rng = rng_for(7000 + cap)
    p = Pair(dev, cap, bits, bucket_count=nb)
    keys = distinct_u64(rng, cap)
    keys[:1] = RESERVED[1]
    vals = rng.integers(0, 1 << 32, size=cap, dtype=np.uint64)
    p.insert(keys, vals.astype(np.uint32) if bits == 32 else vals)
    p.erase(keys[1:cap // 3])
    pool = np.concatenate([keys, distinct_u64(rng, cap), RESERVED])
    for n in SIZES:
        p.find(pool[rng.integers(0, pool.size, size=n)])


@pytest.mark.parametrize("path", [ct.INSERT_SPECULATIVE, ct.INSERT_RESOLVE_FIRST])
@pytest.mark.parametrize("bits", [0, 32, 64])
@pytest.mark.parametrize("cap,nb", TABLES)
def test_insert_erase_batch_sizes(dev, cap, nb, bits, path):  # noqa: F811
    """Batches of every size in SIZES inserted into and erased from tables that fill up, so that
    many keys claim in the same bucket at the same time, wrap around, and meet FULL."""
    rng = rng_for(7100 + cap)
    p = Pair(dev, cap, bits, bucket_count=nb, path=path)
    pool = np.concatenate([distinct_u64(rng, 2 * cap), RESERVED])

    def batch(n):
        k = pool[rng.integers(0, pool.size, size=n)]
        v = rng.integers(0, 1 << 32, size=n, dtype=np.uint64)
        return k, v.astype(np.uint32) if bits == 32 else v

    for r, n in enumerate(SIZES):
        p.insert(*batch(n))
        p.erase(batch(n)[0])
        p.find(batch(n)[0])
        if r % 5 == 0:
            p.g.debug_inject_claim_losses(r % 3)   # every, none or every second first claim lost
        p.g.size()                                 # the host's size bound: provable chunks again
    p.same_state()


@pytest.mark.parametrize("cap,nb", [(64, 8), (104, 13), (4096, 0)])
def test_alloc_release_batch_sizes(dev, cap, nb):  # noqa: F811
    rng = rng_for(7200 + cap)
    p = Pair(dev, cap, 32, hash_kind=ct.HASH_VOXEL21, bucket_count=nb, pool=cap // 2)
    pool = np.concatenate([distinct_u64(rng, cap) >> np.uint64(1), RESERVED])
    for n in SIZES:
        p.insert_alloc(pool[rng.integers(0, pool.size, size=n)])
        p.erase_release(pool[rng.integers(0, pool.size, size=n)])
    p.same_state()
