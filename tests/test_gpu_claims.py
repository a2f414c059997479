"""Lost claims of the batch inserts: keys that crowd into one bucket, so that most claims lose and go
on, and the test hook that makes chosen keys lose.  The hook's losses show in where the keys lie."""
import numpy as np
import pytest
import torch

from test_gpu_parity import PATHS, Pair, dev, g64  # noqa: F401
from test_gpu_partitioned import partitioned
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

M64 = np.uint64(0xFFFFFFFFFFFFFFFF)


def fmix64(k):
    k = k ^ (k >> np.uint64(33))
    k = k * np.uint64(0xFF51AFD7ED558CCD)
    k = k ^ (k >> np.uint64(33))
    k = k * np.uint64(0xC4CEB9FE1A85EC53)
    return k ^ (k >> np.uint64(33))


def scale(mix, n):
    """floor(mix * n / 2^64) for n < 2^31."""
    lo, hi = mix & np.uint64(0xFFFFFFFF), mix >> np.uint64(32)
    return (hi * np.uint64(n) + (lo * np.uint64(n) >> np.uint64(32))) >> np.uint64(32)


def home_and_rot(keys, nb):
    """Home bucket and first slot in order of generic keys, for a prime bucket count."""
    mix = fmix64(keys)
    turned = mix << np.uint64(32) | mix >> np.uint64(32)
    step = np.uint64(1) + scale(turned, nb - 1)
    return scale(mix, nb), step >> np.uint64(1) & np.uint64(7)


def keys_of_bucket(rng, bucket, nb, n):
    """n distinct generic keys with one home bucket: fmix64 turned back from mixes of that bucket."""
    lo, hi = -(-(bucket << 64) // nb), ((bucket + 1) << 64) // nb
    k = np.unique(rng.integers(lo, hi, size=n + 16, dtype=np.uint64))[:n]
    for factor in (0xC4CEB9FE1A85EC53, 0xFF51AFD7ED558CCD):
        k = k ^ (k >> np.uint64(33))
        k = k * np.uint64(pow(factor, -1, 1 << 64))
    k = rng.permutation(k ^ (k >> np.uint64(33)))
    assert k.size == n and (home_and_rot(k, nb)[0] == bucket).all()
    return k


def chosen(keys, every):
    """Keys that the hook makes lose."""
    return (fmix64(keys ^ np.uint64(0x9E3779B97F4A7C15)) >> np.uint64(32)) % np.uint64(every) == 0


def slots_of(t):
    """Keys of the buckets, (bucket, slot): they follow the 256-byte header, 128 bytes each."""
    raw = t.buf[256:256 + t.bucket_count * 128].cpu().numpy().view(np.uint64)
    return raw.reshape(t.bucket_count, 8, 2)[:, :, 0]


def assert_losses(t, keys, every, rot=None, share=4):
    """Every key alone in its home bucket lies in its first slot, or in the next when it lost that."""
    at = slots_of(t)
    home, r = home_and_rot(keys, t.bucket_count)
    rot = r if rot is None else rot
    alone = (np.bincount(home.astype(np.int64), minlength=t.bucket_count)[home.astype(np.int64)] == 1)
    alone &= (at < M64 - np.uint64(1)).sum(axis=1)[home.astype(np.int64)] == 1
    assert alone.sum() > keys.size // share
    want = rot + chosen(keys, every).astype(np.uint64) & np.uint64(7)
    k, h, w = keys[alone], home[alone].astype(np.int64), want[alone].astype(np.int64)
    np.testing.assert_array_equal(at[h, w], k)


# one workgroup (to 2048 keys), reading ahead (to 2^16), beyond
@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("every", [1, 2, 7])
@pytest.mark.parametrize("n", [1, 1500, 5000, 70_001])
def test_injected_losses_take_the_next_slot(dev, n, every, path):  # noqa: F811
    keys = distinct_u64(rng_for(7700, n), n)
    nb = {1: 13, 1500: 4099, 5000: 10_007, 70_001: 140_009}[n]
    p = Pair(dev, 8 * nb, 64, bucket_count=nb, path=path)
    p.g.debug_inject_claim_losses(every)
    batch = np.concatenate([keys, keys[::3]])
    p.insert(batch, np.arange(batch.size, dtype=np.uint64))
    p.same_state()
    assert_losses(p.g, keys, every)
    dst = ct.Table(8 * nb, ct.VAL_U64, bucket_count=nb, device=dev)
    dst.debug_inject_claim_losses(every)
    p.g.rehash_into(dst)
    assert_losses(dst, keys, every)


def test_injected_losses_in_bins(dev):  # noqa: F811
    """The same in an insert that brings the keys to the buckets, where the order is the key's top bits."""
    n, nb, every = 1 << 23, 2_796_181, 2      # three keys per bucket
    keys = distinct_u64(rng_for(7702), n)
    t = ct.Table(8 * nb, ct.VAL_U64, bucket_count=nb, device=dev)
    t.set_insert_path(ct.INSERT_SPECULATIVE)
    assert partitioned(t, n)
    t.debug_inject_claim_losses(every)
    k = g64(keys, dev)
    assert bool((t.insert(k, k) == 1).all())
    v, f = t.find(k)
    assert bool(f.all()) and torch.equal(v, k) and t.size() == n and t.check() == 0
    assert_losses(t, keys, every, keys >> np.uint64(61), 30)


# one workgroup (and a table that cannot hold them all), reading ahead, beyond
@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("every", [0, 1, 2])
@pytest.mark.parametrize("nb,n", [(13, 150), (4099, 3000), (40_009, 70_001)])
def test_keys_of_one_bucket(dev, nb, n, every, path):  # noqa: F811
    """Keys of one home bucket in one batch: a wave's lanes all find its eight slots free, so most lose
    every claim there and go on along their paths.  Then half of them leave and others come into
    the tombstones."""
    rng = rng_for(7701, n)
    crowd = keys_of_bucket(rng, 5, nb, n)
    p = Pair(dev, 8 * nb, 64, bucket_count=nb, path=path)
    p.g.debug_inject_claim_losses(every)
    for part in (crowd[: n // 2], crowd[n // 3:]):
        k = np.concatenate([part, part[::-2]])
        k = k[rng.permutation(k.size)]
        p.g.size()   # the host's size bound: provable chunks where there is room
        p.insert(k, np.arange(k.size, dtype=np.uint64))
        p.same_state()
        p.find(crowd)
        p.erase(crowd[::2])
        p.same_state()
