"""The words that batches count into are zero between batches.  What a batch that failed half way would
leave there (written by the test through the table's buffer) is gone after a clear, and before the
table's next batch, so the live count stays the oracle's."""
import numpy as np
import pytest
import torch

from test_gpu_parity import PATHS, Pair, dev, g64  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu

N = 5000


def leave_counts(t):
    """As if a batch of 3 stored keys per word had not been summed, and 7 had not been settled."""
    words = t.buf[t.nbytes - 4096:].view(torch.int64)
    assert not words[::16].any() and int(words[1]) == 0     # (between them, nothing is used)
    words[::16] = 3 << 32
    words[1] = 7 << 20


def pair(dev, path):  # noqa: F811
    p = Pair(dev, 1 << 16, 64, path=path)
    k = distinct_u64(rng_for(7900), 3 * N)
    p.insert(k[:N], k[:N])
    return p, k


def fail(call):
    """A call that reports a HIP error: that of an invalid device set just before it."""
    assert ct.lib().hipSetDevice(9999) != 0
    assert call() == ct.CT_E_HIP
    torch.cuda.synchronize()


@pytest.mark.parametrize("path", PATHS)
def test_clear_zeroes_counts(dev, path):  # noqa: F811
    p, k = pair(dev, path)
    leave_counts(p.g)
    p.g.clear()
    p.o.clear()
    p.insert(k, k)
    p.erase(k[::2])
    p.same_state()


@pytest.mark.parametrize("op", ["insert", "erase"])
@pytest.mark.parametrize("path", PATHS)
def test_a_failed_batch_leaves_no_counts(dev, path, op):  # noqa: F811
    p, k = pair(dev, path)
    keys = g64(k[N:2 * N], dev)
    fail(lambda: ct.lib().ct_insert_batch(p.g._h, ct._ptr(keys), ct._ptr(keys), N, None, ct._stream(dev)))
    p.o.insert(k[N:2 * N], k[N:2 * N])     # (its launches have run all the same)
    leave_counts(p.g)
    if op == "insert":
        p.insert(k, k)
    else:
        p.erase(k[::2])
    p.same_state()


def test_a_failed_grouped_plan_leaves_no_counts(dev):  # noqa: F811
    p, k = pair(dev, ct.INSERT_SPECULATIVE)
    keys = g64(k, dev)
    plan = ct.Plan(device=dev)
    plan.add(p.g, ct.OP_INSERT, keys=keys, vals=keys)
    plan.group()
    fail(lambda: ct.lib().ct_plan_launch_grouped(plan._h, ct._stream(dev)))   # ends after its first stage
    leave_counts(p.g)
    plan.launch_grouped()
    p.o.insert(k, k)
    p.same_state()
