"""Entries of neighbouring tiles leave as one run, also where each tile is of another tensor and its entries are numbered by
themselves: tensors of less than a tile, of one tile, of two and of several in one bucket, little and much changed, buckets
that hold everything and buckets that end in the middle of a run."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import Case, full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import T
from test_gpu_refresh import check_refresh
from workloads import synth

pytestmark = pytest.mark.gpu

TILE = 8192
# elements a shard: halves, single elements, whole tiles, tiles and one more, several tiles between
SIZES = [TILE // 2] * 60 + [1, TILE, 7] * 20 + [TILE] * 90 + [TILE + 1, 3 * TILE, TILE - 1, 9 * TILE] * 12 + [2 * TILE] * 40 + [100] * 150


def make(tp, p, fp32, **kw):
    ts = [T(tp, n, R.SPLIT_ROWS) for n in SIZES]
    olds, news = [], []
    for _, _, o, n in synth.model_pairs(ts, "bernoulli", 23, "cpu", p=p):
        olds.append(o)
        news.append(n.float() if fp32 else n)
    return Case(ts, tp, olds, news, **kw)


@pytest.mark.parametrize("what", ["new", "arith", "refresh", "arith refresh"])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("tp,p", [(1, 0.01), (3, 0.05), (2, 0.3)])
def test_tiles_of_many_tensors(tp, p, fp32, what, tile_order):
    print("case: runs of tiles tp=%d p=%g fp32=%s %s order=%d" % (tp, p, fp32, what, tile_order), flush=True)
    c = make(tp, p, fp32)
    if what == "new":
        full_parity(c, check_dense=False)
    elif what == "refresh":
        check_refresh(c)
    else:
        check_arith(c, R.ENCODE_ARITH | (R.ENCODE_REFRESH if what == "arith refresh" else 0))


@pytest.mark.parametrize("room", [0.3, 0.77])
def test_bucket_ends_in_a_run(room, tile_order):
    print("case: a bucket ends in a run, room for %g, order=%d" % (room, tile_order), flush=True)
    c = make(2, 0.02, False, capacity=16)
    want = oracle.encode_model(c.records(), 2)
    guard, caps = 4096, [int(w["seg_off"][-1] * room) for w in want]
    for b, cap in zip(c.buckets, caps):
        b.capacity = cap
        b.idx = torch.full((cap + guard,), -7, dtype=torch.int32, device="cuda")
        b.val = torch.full((cap + guard,), -7, dtype=torch.int16, device="cuda")
    c.encode()
    for d, (b, cap) in enumerate(zip(c.buckets, caps)):
        with pytest.raises(R.RoseError) as e:
            R.bucket_check(c.plan, b)
        assert e.value.required == want[d]["seg_off"][-1]
        assert np.array_equal(b.seg_off.cpu().numpy(), want[d]["seg_off"])
        assert np.array_equal(b.idx[:cap].cpu().numpy(), want[d]["idx"][:cap])
        assert np.array_equal(b.val[:cap].cpu().numpy().view(np.uint16), want[d]["val"][:cap])
        assert (b.idx[cap:] == -7).all() and (b.val[cap:] == -7).all()
