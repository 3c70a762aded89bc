"""The order check of a transport object: one entry that does not exceed the one before it turns the object away
unless a tensor's entries begin there, wherever in the check's work (a lane's four entries, a wave's 256, a
workgroup's 1024 or 4096) it stands, and however many tensors begin nearby."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


def make(sizes, p, seed):
    """An object of every size's entries, as bytes on the host, and where its arrays lie."""
    rng = np.random.default_rng(seed)
    plan = R.shard_plan([T(1 if n else 0, max(n, 1), R.REPLICATED) for n in sizes], 1)
    plan.upload()
    idx, seg = [], [0]
    for n in sizes:
        hit = np.flatnonzero(rng.random(n) < p).astype(np.int32)
        idx.append(hit)
        seg.append(seg[-1] + hit.size)
    idx = np.concatenate(idx)
    b = R.Bucket(seg[-1], len(sizes))
    b.idx[:seg[-1]] = torch.from_numpy(idx).cuda()
    b.val[:seg[-1]] = torch.from_numpy(rng.integers(1, 1 << 15, size=seg[-1], dtype=np.int16)).cuda()
    b.seg_off.copy_(torch.tensor(seg, dtype=torch.int64))
    obj = torch.empty(R.object_bytes(plan, seg[-1]), dtype=torch.uint8, device="cuda")
    R.bucket_pack(plan, 0, b, 0, seg[-1], obj)
    at = (64 + 8 * (len(sizes) + 1) + 15) & ~15
    return plan, obj, obj[at:at + 4 * seg[-1]].view(torch.int32), np.array(seg)


def applied(plan, obj, sizes):
    flat = torch.zeros(sum(sizes) + 1, dtype=torch.int16, device="cuda")
    views, at = [], 0
    for n in sizes:
        views.append(flat[at:at + max(n, 1)])
        at += n
    R.object_apply(plan, obj, R.ptr_table(views))
    torch.cuda.synchronize()
    return int(torch.count_nonzero(flat))


@pytest.mark.parametrize("name,sizes,p", [("threes", [3] * 1500, 1.0), ("holes", ([9] + [0] * 70) * 300, 0.9),
                                          ("hundreds", [100, 1, 700, 65] * 60, 0.3), ("two", [40000, 30000], 0.2),
                                          ("large", [1 << 20, 1 << 20, 300000, 7], 1.0)])
def test_one_entry_out_of_order(name, sizes, p):
    print("case: object check %s" % name, flush=True)
    plan, obj, idx, seg = make(sizes, p, seed=len(sizes))
    n = int(seg[-1])
    assert applied(plan, obj, sizes) == n, "an object in order was turned away"
    starts = set(seg.tolist())
    places = sorted({x for c in (1, 4, 255, 256, 257, 1023, 1024, 1025, 4095, 4096, n // 2, n - 1) for x in (c, c + 1)
                     if 0 < x < n and x not in starts})
    assert len(places) > 5
    for x in places:
        keep = idx[x].clone()
        idx[x] = idx[x - 1]                             # no longer above the entry before it
        assert applied(plan, obj, sizes) == 0, x
        idx[x] = keep
    assert applied(plan, obj, sizes) == n


def test_segment_table_out_of_order():
    print("case: object check, tables", flush=True)
    sizes = [50] * 40
    plan, obj, idx, seg = make(sizes, 0.5, seed=1)
    table = obj[64:64 + 8 * len(seg)].view(torch.int64)
    for t, v in [(3, int(seg[5])), (7, -1), (20, int(seg[-1]) + 1), (39, 1 << 62), (12, -(1 << 62))]:
        keep = table[t].clone()
        table[t] = v
        assert applied(plan, obj, sizes) == 0, (t, v)
        table[t] = keep
    assert applied(plan, obj, sizes) == int(seg[-1])


@pytest.mark.parametrize("n", [1, 3, 4, 7, 8, 9, 1023, 1024, 1025, 2047, 4097, (1 << 21) - 1, (1 << 21) + 1, (1 << 21) + 4099])
@pytest.mark.parametrize("first", [0, 1, 6])
def test_packed_ranges(n, first):
    """The object's arrays are the bucket's range, at the edges of a lane's, a workgroup's and a launch's share."""
    print("case: pack n=%d first=%d" % (n, first), flush=True)
    total = n + first + 2
    plan = R.shard_plan([T(1, total, R.REPLICATED)], 1)
    b = R.Bucket(total, 1)
    b.idx[:total] = torch.arange(total, dtype=torch.int32, device="cuda")
    b.val[:total] = torch.randint(-30000, 30000, (total,), device="cuda", dtype=torch.int16)
    b.seg_off.copy_(torch.tensor([0, total], dtype=torch.int64))
    size = R.object_bytes(plan, n)
    store = torch.full((size + 64,), 0xEE, dtype=torch.uint8, device="cuda")
    R.bucket_pack(plan, 0, b, first, n, store[:size])
    torch.cuda.synchronize()
    a, v = 80, 80 + (4 * n + 15) // 16 * 16
    assert torch.equal(store[a:a + 4 * n].view(torch.int32), b.idx[first:first + n])
    assert torch.equal(store[v:v + 2 * n].view(torch.int16), b.val[first:first + n])
    assert not store[a + 4 * n:v].any() and not store[v + 2 * n:size].any() and (store[size:] == 0xEE).all()
