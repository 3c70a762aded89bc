"""The slack of a transport object is zero whatever the memory held: the 8 bytes between the segment table and the indices
(there for even numbers of tensors), behind the indices and behind the values; also of an object of a range that the bucket
does not hold, which nobody applies."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tensors", [1, 2, 4, 300])
@pytest.mark.parametrize("n", [0, 1, 7, 1000, (1 << 21) + 33])
def test_slack_is_zero(n, n_tensors):
    print("case: object slack, %d entries, %d tensors" % (n, n_tensors), flush=True)
    room = n + 50
    plan = R.shard_plan([T(1, room, R.REPLICATED)] * n_tensors, 1)
    b = R.Bucket(room, n_tensors)
    g = np.random.default_rng(n_tensors)
    idx = g.integers(0, 1 << 31, room, dtype=np.int64).astype(np.int32)
    val = g.integers(0, 1 << 16, room, dtype=np.int64).astype(np.uint16)
    seg = np.sort(g.integers(0, room, n_tensors + 1))
    seg[0], seg[-1] = 0, room
    b.idx.copy_(torch.from_numpy(idx))
    b.val.copy_(torch.from_numpy(val.view(np.int16)))
    b.seg_off.copy_(torch.from_numpy(seg))
    size = R.object_bytes(plan, n)
    store = torch.full((size + 128,), 0xEE, dtype=torch.uint8, device="cuda")
    R.bucket_pack(plan, 0, b, 3, n, store[64:64 + size])
    got = store.cpu().numpy()
    want = oracle.pack_object({"idx": idx, "val": val, "seg_off": seg}, 0, 3, n)
    assert np.array_equal(got[64:64 + size], want)
    assert (got[:64] == 0xEE).all() and (got[64 + size:] == 0xEE).all()
    b.seg_off[-1] = n + 2                                # one entry short of the range
    store.fill_(0xEE)
    R.bucket_pack(plan, 0, b, 3, n, store[64:64 + size])
    got = store.cpu().numpy()[64:64 + size]
    at = 64 + 8 * (n_tensors + 1)
    assert (got[:4] == 0).all() and (got[at:(at + 15) // 16 * 16] == 0).all()
