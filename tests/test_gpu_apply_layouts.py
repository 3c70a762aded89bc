"""Apply into shards packed one tensor behind the other from any element on, in every way a bucket is
walked (few entries, lines, crowded lines, dense; sized tightly or for everything), with entries and
neighbours compared bit for bit with plain assignment (arithmetic payloads: torch's bf16 addition)."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

# many small tensors (several to a 64-byte line, several segments to a chunk), odd sizes, and large ones
SIZES = [1, 2, 7, 8, 9, 31, 32, 33, 3, 5, 300001, 64, 1, 40000, 65537, 15, 1, 1, 1, 8191]


@pytest.mark.parametrize("p", [0.002, 0.01, 0.05, 0.12, 0.3, 1.0])
@pytest.mark.parametrize("first", [0, 1, 5, 8, 24, 31])
@pytest.mark.parametrize("payload", ["new", "arith"])
@pytest.mark.parametrize("many", [False, True])
def test_packed_shard(p, first, payload, many):
    print("case: packed apply p=%g first=%d %s many=%s" % (p, first, payload, many), flush=True)
    sizes = SIZES + [3] * 600 + [100003] if many else SIZES      # more than 512 segments: the other search
    rng = np.random.default_rng(int(p * 1000) + first)
    plan = R.shard_plan([T(1, n, R.REPLICATED) for n in sizes], 1)
    plan.upload()
    total = sum(sizes)
    flat = rng.integers(0x3C00, 0x3F80, size=total + first + 40, dtype=np.uint16)
    want = flat.copy()
    idx, val, seg, at = [], [], [0], first
    for n in sizes:
        hit = np.flatnonzero(rng.random(n) < p).astype(np.int32)
        v = rng.integers(0x3C00, 0x3F80, size=hit.size, dtype=np.uint16)
        esc = rng.random(hit.size) < 0.3 if payload == "arith" else np.ones(hit.size, bool)
        was = torch.from_numpy(want[at + hit].view(np.int16)).view(torch.bfloat16)
        added = (was + torch.from_numpy(v.view(np.int16)).view(torch.bfloat16)).view(torch.int16).numpy().view(np.uint16)
        want[at + hit] = np.where(esc, v, added)
        idx.append(np.where(esc, hit | np.int32(-2 ** 31), hit) if payload == "arith" else hit)
        val.append(v)
        seg.append(seg[-1] + hit.size)
        at += n
    for capacity in (max(seg[-1], 1), total):
        b = R.Bucket(capacity, len(sizes))
        b.idx[:seg[-1]] = torch.from_numpy(np.concatenate(idx).astype(np.int32)).cuda()
        b.val[:seg[-1]] = torch.from_numpy(np.concatenate(val).view(np.int16)).cuda()
        b.seg_off.copy_(torch.tensor(seg, dtype=torch.int64))
        dst = torch.from_numpy(flat.view(np.int16).copy()).cuda()
        assert dst.data_ptr() % 64 == 0
        views, at = [], first
        for n in sizes:
            views.append(dst[at:at + n])
            at += n
        R.delta_apply_ex(plan, 0, b, R.PAYLOAD_ARITH if payload == "arith" else R.PAYLOAD_NEW, R.ptr_table(views))
        torch.cuda.synchronize()
        assert np.array_equal(dst.cpu().numpy().view(np.uint16), want)


def test_odd_address():
    """A destination at an odd byte address has no elements in lines."""
    n = 5000
    plan = R.shard_plan([T(1, n, R.REPLICATED)], 1)
    plan.upload()
    b = R.Bucket(n, 1)
    hit = torch.arange(0, n, 7, dtype=torch.int32, device="cuda")
    b.idx[:hit.numel()] = hit
    b.val[:hit.numel()] = torch.arange(hit.numel(), dtype=torch.int16, device="cuda")
    b.seg_off.copy_(torch.tensor([0, hit.numel()], dtype=torch.int64))
    raw = torch.zeros(2 * n + 64, dtype=torch.uint8, device="cuda")
    R.delta_apply(plan, 0, b, torch.tensor([raw.data_ptr() + 1], dtype=torch.int64, device="cuda"))
    torch.cuda.synchronize()
    want = torch.zeros(n, dtype=torch.int16)
    want[::7] = torch.arange(hit.numel(), dtype=torch.int16)
    got = raw.cpu().numpy()
    assert np.array_equal(got[1:1 + 2 * n].view(np.int16), want.numpy()) and got[0] == 0 and not got[1 + 2 * n:].any()
