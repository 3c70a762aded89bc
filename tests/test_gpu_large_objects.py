"""Objects of more than 2 M entries, whose arrays are copied by lines of the object: byte-identical to the oracle's wherever
the object's arrays and the range in the bucket begin, for lengths around whole tiles of 4096 entries."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

FEW = 1 << 21


@pytest.mark.parametrize("n_tensors", [1, 3, 9])
@pytest.mark.parametrize("more", [1, 31, 32, 63, 64, 4095, 4096, 4097, 4096 + 40])
def test_large_objects(more, n_tensors):
    print("case: large object of 2 M + %d, %d tensors" % (more, n_tensors), flush=True)
    n, spare = FEW + more, 10000
    plan = R.shard_plan([T(1, n + spare, R.REPLICATED)] * n_tensors, 1)
    b = R.Bucket(n + spare, n_tensors)
    g = np.random.default_rng(more)
    idx = g.integers(0, 1 << 31, n + spare, dtype=np.int64).astype(np.int32)
    val = g.integers(0, 1 << 16, n + spare, dtype=np.int64).astype(np.uint16)
    seg = np.sort(g.integers(0, n + spare, n_tensors + 1))
    seg[0], seg[-1] = 0, n + spare
    b.idx.copy_(torch.from_numpy(idx))
    b.val.copy_(torch.from_numpy(val.view(np.int16)))
    b.seg_off.copy_(torch.from_numpy(seg))
    size = R.object_bytes(plan, n)
    store = torch.empty(size + 512, dtype=torch.uint8, device="cuda")
    for first, at in [(0, 0), (1, 16), (5, 112), (spare, 64)]:
        store.fill_(0xEE)
        R.bucket_pack(plan, 0, b, first, n, store[128 + at:128 + at + size])
        got = store.cpu().numpy()
        assert np.array_equal(got[128 + at:128 + at + size], oracle.pack_object({"idx": idx, "val": val, "seg_off": seg}, 0, first, n))
        assert (got[:128 + at] == 0xEE).all() and (got[128 + at + size:] == 0xEE).all()
