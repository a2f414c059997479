"""Merged runs copy operations of any size from and to arrays of any alignment: nothing outside an
operation's arrays changes, and results equal the single-table calls'."""
import numpy as np
import pytest
import torch

from test_gpu_multi import dev, g32, g64  # noqa: F401
from paper_1908_05936_amd import ct
from paper_1908_05936_amd.workloads import distinct_u64, rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1, 1, 2, 3, 5], [15, 16, 17, 31, 1], [4097, 1, 16385, 255, 70000]])
@pytest.mark.parametrize("gap", [0, 1, 7])
def test_merged_copies(dev, sizes, gap):  # noqa: F811
    rng = rng_for(7500, gap)
    n = sum(sizes)
    keys = distinct_u64(rng, n)
    keys[n // 2:] = keys[rng.integers(0, n // 2 + 1, size=n - n // 2)]   # present and repeated ones
    vals = rng.integers(0, 1 << 31, size=n, dtype=np.uint32)
    t = ct.Table(2 * n + 8, ct.VAL_U32, chunk=1 << 17, device=dev)
    one = ct.Table(2 * n + 8, ct.VAL_U32, device=dev)
    k, v = g64(keys, dev), g32(vals, dev)
    total = n + gap * (len(sizes) + 1)
    ins, fnd = (torch.full((total,), 0xAA, dtype=torch.uint8, device=dev) for _ in range(2))
    out = torch.full((total,), -7, dtype=torch.int32, device=dev)
    p = ct.Plan(dev)
    keep = torch.zeros(total, dtype=torch.bool, device=dev)
    for op in (ct.OP_INSERT, ct.OP_FIND):
        at, pos = gap, 0
        for b in sizes:
            s, d = slice(pos, pos + b), slice(at, at + b)
            keep[d] = True
            if op == ct.OP_INSERT:
                p.add(t, op, k[s], vals=v[s], flags_out=ins[d])
            else:
                p.add(t, op, k[s], vals_out=out[d], flags_out=fnd[d])
            at, pos = at + b + gap, pos + b
    p.group(merge_runs=True)
    p.launch_grouped()
    est = one.insert(k, v)
    ev, ef = one.find(k)
    assert torch.equal(ins[keep], est) and torch.equal(fnd[keep], ef) and torch.equal(out[keep], ev)
    assert bool((ins[~keep] == 0xAA).all()) and bool((fnd[~keep] == 0xAA).all()) and bool((out[~keep] == -7).all())
    assert t.check() == 0
