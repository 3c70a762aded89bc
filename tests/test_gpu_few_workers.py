"""Much comes, few workers walk, and chains end in short blocks: a worker that has counted the rest of its ticket ahead gets a
second ticket of the same group, which has no tile in such a block.  Same buckets as ever (tests/sanitize/walk_driver.cpp walks
such shapes on the CPU)."""
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import assert_buckets_equal, bits
from test_gpu_pipeline import cut, dev, model
from workloads import models, synth

pytestmark = pytest.mark.gpu


def check_arith(ts, recs, plan, buckets, tp):
    """Arithmetic payloads applied to the receivers' previous weights give their new ones."""
    for b, bucket in enumerate(buckets):
        R.bucket_check(plan, bucket)
        dst = [dev(cut(r["old"], r, tp, b % tp)) for r in recs]
        R.delta_apply_ex(plan, b, bucket, R.PAYLOAD_ARITH, R.ptr_table(dst))
        torch.cuda.synchronize()
        for i, r in enumerate(recs):
            if plan.local_numel(i, b) > 0:
                assert (bits(dst[i]) == cut(r["new"], r, tp, b % tp)).all(), "bucket %d tensor %d" % (b, i)


# chains of 158 tiles; long chains of a model at TP4 and in three stages; a sender's long chain between short ones
SHAPES = [(3, 1, 0, 1, 70, 0.4), (3, 1, 0, 1, 66, 0.6), (4, 1, 0, 1, 0, 0.4), (1, 1, 0, 3, 0, 0.4), (4, 4, 2, 1, 80, 0.6)]
# (arithmetic payloads are checked by applying them, which takes all of a receiver's senders)
CASES = [x + y for x in SHAPES for y in [(False, False), (True, False), (False, True)] if not (x[1] > 1 and y[0])]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("tp,tp_src,src,pp_dst,workers,p,arith,refresh", CASES)
def test_much_and_short_chains(tp, tp_src, src, pp_dst, workers, p, arith, refresh, f32, tile_order):
    print("case: much and short chains, tp %d of %d rank %d, %d stages, %d workers, p %g, f32 %d, arith %d, refresh %d, order %d" % (
        tp, tp_src, src, pp_dst, workers, p, f32, arith, refresh, tile_order), flush=True)
    n_layers = 6
    if tp == 3:
        ts = models.decoder(n_layers, 192, 6, 3, 32, 576, 1536, fused=True)
        recs = [dict(t, old=bits(o), new=bits(n)) for _, t, o, n in synth.model_pairs(ts, "bernoulli", 18, "cpu", p=p)]
    else:
        ts, recs = model(n_layers, seed=18, p=p)
    plan = R.binding.shard_plan(ts, tp, tp_src, src, n_layers, 1, 0, pp_dst)
    if workers:
        plan.set_worker_cap(workers)
    sl = [dict(r, old=cut(r["old"], r, tp_src, src), new=cut(r["new"], r, tp_src, src)) for r in recs]
    olds = [dev(x["old"]) for x in sl]
    news = [(dev(x["new"]).to(torch.int32) << 16).view(torch.float32) if f32 else dev(x["new"]) for x in sl]
    buckets = [R.Bucket(plan.bucket_capacity(b) * 7 // 10 + 64, len(ts)) for b in range(plan.n_buckets)]
    dtype, ws = R.FP32_RNE if f32 else R.BF16, R.workspace(plan)
    if refresh:
        R.delta_encode_refresh(plan, R.ptr_table(olds), R.ptr_table(news), dtype, buckets, ws)
    else:
        R.delta_encode_ex(plan, R.ptr_table(olds), R.ptr_table(news), dtype, R.ENCODE_ARITH if arith else 0, buckets, ws)
    torch.cuda.synchronize()
    if arith:
        return check_arith(ts, recs, plan, buckets, tp)
    want = oracle.encode_model_pp(sl, tp, tp_src, src, n_layers, 1, 0, pp_dst)
    for b in range(plan.n_buckets):
        n = R.bucket_check(plan, buckets[b])
        got = {"idx": buckets[b].idx[:n].cpu().numpy(), "val": buckets[b].val[:n].cpu().numpy().view("uint16"),
               "seg_off": buckets[b].seg_off.cpu().numpy()}
        assert_buckets_equal(got, want[b], "bucket %d" % b)
    for i, (o, x) in enumerate(zip(olds, sl)):
        if refresh:
            assert (bits(o) == x["new"]).all(), "tensor %d not refreshed" % i
