"""Apply on both sides of the lines its launch is chosen by: small workgroups or large (8192 chunks of 64
entries), sparse or not (room for a 24th of the shard), five waves a SIMD or eight (a 20th), twice the workgroups or not (a third of it).  Bucket and
object, compared bit for bit with plain assignment."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

SMALL = 8192 * 64


@pytest.mark.parametrize("capacity", [1, 255, 257, SMALL - 1, SMALL, SMALL + 1, SMALL + 511])
@pytest.mark.parametrize("times", [1, 3, 4, 22, 25])
@pytest.mark.parametrize("fill", [0.2, 1.0])
def test_lines_of_the_launch(capacity, times, fill):
    print("case: apply launch capacity=%d shard=%d x fill=%g" % (capacity, times, fill), flush=True)
    rng = np.random.default_rng(capacity % 1000 + times)
    numel = capacity * times
    sizes = [numel // 3, numel - numel // 3] if numel > 2 else [0, numel]
    plan = R.shard_plan([T(1 if n else 0, max(n, 1), R.REPLICATED) for n in sizes], 1)
    plan.upload()
    total = max(1, int(capacity * fill))
    hit = np.sort(rng.permutation(numel)[:total]) if times > 1 or fill < 1 else np.arange(total)
    val = rng.integers(0, 1 << 16, size=total, dtype=np.uint16)
    flat = rng.integers(0, 1 << 16, size=numel + 3, dtype=np.uint16)
    want = flat.copy()
    want[3 + hit] = val
    split = int(np.searchsorted(hit, sizes[0]))
    b = R.Bucket(capacity, 2)
    b.idx[:total] = torch.from_numpy(np.where(hit < sizes[0], hit, hit - sizes[0]).astype(np.int32)).cuda()
    b.val[:total] = torch.from_numpy(val.view(np.int16)).cuda()
    b.seg_off.copy_(torch.tensor([0, split, total], dtype=torch.int64))
    dst = torch.from_numpy(flat.view(np.int16).copy()).cuda()
    R.delta_apply(plan, 0, b, R.ptr_table([dst[3:3 + sizes[0]], dst[3 + sizes[0]:]]))
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), want), "bucket"
    obj = torch.empty(R.object_bytes(plan, total), dtype=torch.uint8, device="cuda")
    R.bucket_pack(plan, 0, b, 0, total, obj)
    dst = torch.from_numpy(flat.view(np.int16).copy()).cuda()
    R.object_apply(plan, obj, R.ptr_table([dst[3:3 + sizes[0]], dst[3 + sizes[0]:]]))
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), want), "object"
