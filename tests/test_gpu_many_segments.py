"""Chunks of a bucket that hold entries of many tensors: every lane finds its own segment (fewer than 64 of them
ahead, exactly 64, more, empty ones between), a line that the chunk shares with the one before or behind it is
written once.  Buckets and objects, tensors right behind each other from an odd element on; the receiver's shard
is compared bit for bit with plain assignment."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from gpu_harness import full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import T
from test_gpu_refresh import check_refresh
from test_gpu_unaligned import packed_case

pytestmark = pytest.mark.gpu

SIZES = {"threes": [3] * 1500, "ones": [1] * 700, "forties": [40] * 900, "hundreds": [100, 1, 700, 65] * 60,
         "holes": ([2] + [0] * 70) * 40, "one behind": [5000] + [1] * 63 + [5000]}


@pytest.mark.parametrize("payload", [R.PAYLOAD_NEW, R.PAYLOAD_ARITH])
@pytest.mark.parametrize("p", [0.01, 0.1, 0.5, 1.0])
@pytest.mark.parametrize("name", sorted(SIZES))
def test_many_segments(name, p, payload):
    print("case: many segments %s p=%g payload=%d" % (name, p, payload), flush=True)
    sizes, first = SIZES[name], 5
    rng = np.random.default_rng(len(sizes) + int(100 * p))
    plan = R.shard_plan([T(1 if n else 0, max(n, 1), R.REPLICATED) for n in sizes], 1)
    plan.upload()
    flat = rng.integers(0x3C00, 0x3F80, size=sum(sizes) + first + 40, dtype=np.uint16)
    want, idx, val, seg, at = flat.copy(), [], [], [0], first
    for n in sizes:
        hit = np.flatnonzero(rng.random(n) < p).astype(np.int32)
        v = rng.integers(0x3C00, 0x3F80, size=hit.size, dtype=np.uint16)
        was = torch.from_numpy(want[at + hit].view(np.int16)).view(torch.bfloat16)
        added = (was + torch.from_numpy(v.view(np.int16)).view(torch.bfloat16)).view(torch.int16).numpy().view(np.uint16)
        want[at + hit] = added if payload == R.PAYLOAD_ARITH else v
        idx.append(hit)
        val.append(v)
        seg.append(seg[-1] + hit.size)
        at += n
    total = seg[-1]
    b = R.Bucket(total + 9, len(sizes))
    b.idx[:total] = torch.from_numpy(np.concatenate(idx)).cuda()
    b.val[:total] = torch.from_numpy(np.concatenate(val).view(np.int16)).cuda()
    b.seg_off.copy_(torch.tensor(seg, dtype=torch.int64))

    def shard():
        dst = torch.from_numpy(flat.view(np.int16).copy()).cuda()
        out, at = [], first
        for n in sizes:
            out.append(dst[at:at + n] if n else dst[:1])
            at += n
        return dst, R.ptr_table(out)

    dst, tab = shard()
    R.delta_apply_ex(plan, 0, b, payload, tab)
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), want), "bucket"
    dst, tab = shard()
    cuts = sorted({min(c, total) for c in (0, 1, 64, 65, 127, total // 2, total)})
    for a, e in zip(cuts[:-1], cuts[1:]):
        obj = torch.empty(R.object_bytes(plan, e - a), dtype=torch.uint8, device="cuda")
        R.bucket_pack_ex(plan, 0, b, payload, a, e - a, obj)
        R.object_apply(plan, obj, tab)
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), want), "objects"


@pytest.mark.parametrize("run", [1, 5, 8, 40, 700])
@pytest.mark.parametrize("fp32", [False, True])
def test_many_small_tensors_encoded(run, fp32):
    """Tiles of which a few vectors hold anything: contiguous tensors and column blocks, 0 to 700 elements."""
    print("case: many small tensors run=%d fp32=%s" % (run, fp32), flush=True)
    ts = []
    for i in range(40):
        ts += [T(1, run + i % 9, R.REPLICATED), T(1 + i % 3, 2 * run, R.SPLIT_COLS), T(0, 16, R.SPLIT_ROWS), T(2, 9 * run, R.SPLIT_ROWS)]
    full_parity(packed_case(ts, 2, 0.4, run, 1, 3, fp32))
    check_arith(packed_case(ts, 2, 0.4, run + 1, 1, 3, fp32))
    check_refresh(packed_case(ts, 2, 0.4, run + 2, 1, 3, fp32))
