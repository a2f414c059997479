"""Partitioned inserts whose fine bins leave over more elements than their lists hold: copies of keys
whose home bucket is full, some of them listed and some marked, some past the room of the bin."""
import numpy as np
import pytest

from test_gpu_claims import home_and_rot, keys_of_bucket
from test_gpu_parity import Pair, dev  # noqa: F401
from test_gpu_partitioned import N, partitioned
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

BIN = 256          # buckets of a fine bin
LEFT = 512         # left-over elements that a bin's list holds


def room(n, nb):
    """Elements that a fine bin holds."""
    mean = n / nb * BIN
    return min(int(mean + 8.0 * mean ** 0.5) + 64, 2560)


def batch(nb, n, copies):
    """Nine keys of one bucket to insert first, and a batch that repeats the ninth and an absent key."""
    rng = rng_for(7800, copies)
    crowd = keys_of_bucket(rng, nb // 2, nb, 10)
    others = distinct_u64(rng, n - 2 * copies, exclude=crowd)
    k = np.concatenate([others, np.repeat(crowd[8:], copies)])
    return crowd, k[rng.permutation(n)]


# (buckets, copies of each key, whether the bin has room for all of them)
CASES = [(2_796_181, 600, False), (2_796_181, 1500, False), (1_118_519, 180, True)]


@pytest.mark.parametrize("every", [0, 2])
@pytest.mark.parametrize("nb,copies,fits", CASES)
def test_more_left_over_than_a_list_holds(dev, nb, copies, fits, every):  # noqa: F811
    crowd, k = batch(nb, N, copies)
    home = home_and_rot(k, nb)[0].astype(np.int64)
    mine = np.bincount(home[home // BIN == nb // 2 // BIN] % BIN, minlength=BIN)
    assert (mine.sum() <= room(N, nb)) == fits
    left = np.maximum(mine - 8, 0).sum() + min(8, 2 * copies)   # (the full bucket leaves all of its own over)
    assert left * min(1.0, room(N, nb) / mine.sum()) > 1.1 * LEFT
    p = Pair(dev, 8 * nb, 64, bucket_count=nb, path=ct.INSERT_SPECULATIVE)
    p.insert(crowd[:8], np.arange(8, dtype=np.uint64))      # the bucket is full,
    p.insert(crowd[8:9], np.arange(8, 9, dtype=np.uint64))  # so this one lies elsewhere
    p.g.debug_inject_claim_losses(every)
    assert partitioned(p.g, N)
    p.insert(k, np.arange(100, N + 100, dtype=np.uint64))
    p.same_state()
    p.find(crowd)
    p.erase(crowd[8:])
    p.find(crowd)

