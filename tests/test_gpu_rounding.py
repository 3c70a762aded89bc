"""The fp32 -> bf16 rounding of the kernels (a conversion instruction, two values at a time) against the oracle's, on
every upper half of a pattern (all exponents, infinities, NaNs, subnormals) with the lower halves where rounding turns,
in both places of a pair."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
def test_every_upper_half(shift):
    print("case: rounding shift=%d" % shift, flush=True)
    high = np.arange(1 << 16, dtype=np.uint32) << 16
    low = np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], dtype=np.uint32)
    bits = (high[:, None] | low[None, :]).ravel()
    bits = np.concatenate([np.zeros(shift, np.uint32), bits])
    bits = np.concatenate([bits, np.zeros(-bits.size % 8, np.uint32)])
    new = torch.from_numpy(bits.view(np.int32)).cuda()
    plan = R.shard_plan([{"rows": 1, "cols": bits.size, "rule": R.REPLICATED}], 1)
    dst = torch.zeros(bits.size, dtype=torch.int16, device="cuda")
    R.dense_copy(plan, 0, R.ptr_table([new]), R.FP32_RNE, R.ptr_table([dst]))
    old = torch.zeros(bits.size, dtype=torch.int16, device="cuda")
    b = R.Bucket(bits.size, 1)
    R.delta_encode_refresh(plan, R.ptr_table([old]), R.ptr_table([new]), R.FP32_RNE, [b], R.workspace(plan))
    torch.cuda.synchronize()
    want = oracle.rne_bf16(bits)
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), want)
    n = R.bucket_check(plan, b)
    where = np.flatnonzero(want)
    assert n == where.size and np.array_equal(b.idx[:n].cpu().numpy(), where)
    assert np.array_equal(b.val[:n].cpu().numpy().view(np.uint16), want[where])
