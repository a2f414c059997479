"""The wave-cooperative probe round at the sizes where it can go wrong: batches around the lanes of
a wave (64), of a packed round (32, 16, 8) and of a group, on tables of one bucket and up, in every
probe-step mode, with full buckets and tombstones.  Against the oracle, bit exact."""
import numpy as np
import pytest

from test_gpu_parity import RESERVED, Pair, dev  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 255, 256, 257, 1000]
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
