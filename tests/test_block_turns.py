"""Refreshes walk the blocks of equally long chains in turn: the order itself on the CPU, and the kernels on senders whose chains
are of equal and of unequal length."""
import os
import subprocess
import tempfile

import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import assert_buckets_equal, bits
from test_gpu_pipeline import cut, dev, model
from test_host_sanitizers import ROOT, SAN, run
from workloads import models, synth


def test_every_block_once_and_each_chain_in_order():
    csrc = os.path.join(ROOT, "paper_2605_06534_amd", "csrc")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "turns_driver")
        subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN +
                              ["-I", os.path.join(ROOT, "include"), "-I", csrc,
                               os.path.join(ROOT, "tests", "sanitize", "turns_driver.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe])
        run(exe)


# equal chains (tp 4, tp 8); stages of unequal length (the last holds the head); a long and several short ones; two long ones
# between short ones.  With a cap on workers, and in the spread order, refreshes walk chain by chain; the workspace's word 6 says
# from bit 8 on how many chains took turns.
@pytest.mark.gpu
@pytest.mark.parametrize("tp,tp_src,src,pp_dst,workers,turns", [(4, 1, 0, 1, 0, 4), (8, 1, 0, 1, 0, 8), (1, 1, 0, 3, 0, 3), (2, 1, 0, 2, 0, 4),
                                                                (4, 4, 2, 1, 0, 0), (8, 4, 1, 1, 0, 2), (4, 1, 0, 1, 70, 0)])
def test_refresh_in_turns(tp, tp_src, src, pp_dst, workers, turns, tile_order):
    print("case: refresh in turns, tp %d of %d rank %d, %d stages, %d workers, order %d" % (tp, tp_src, src, pp_dst, workers, tile_order), flush=True)
    n_layers = 6
    ts, recs = model(n_layers, seed=17, p=0.05)
    if tp > tp_src > 1:                                # (a tile for each tensor in every chain: larger ones, for long chains to be long)
        ts = models.decoder(n_layers, 512, 16, 8, 32, 1408, 1024, fused=True)
        recs = [dict(t, old=bits(o), new=bits(n)) for _, t, o, n in synth.model_pairs(ts, "bernoulli", 17, "cpu", p=0.05)]
    plan = R.binding.shard_plan(ts, tp, tp_src, src, n_layers, 1, 0, pp_dst)
    if workers:
        plan.set_worker_cap(workers)
    sl = [dict(r, old=cut(r["old"], r, tp_src, src), new=cut(r["new"], r, tp_src, src)) for r in recs]
    olds, news = [dev(x["old"]) for x in sl], [dev(x["new"]) for x in sl]
    buckets = [R.Bucket(plan.bucket_capacity(b) * 7 // 100 + 64, len(ts)) for b in range(plan.n_buckets)]
    ws = R.workspace(plan)
    R.delta_encode_refresh(plan, R.ptr_table(olds), R.ptr_table(news), R.BF16, buckets, ws)
    torch.cuda.synchronize()
    assert int(ws.view(torch.int32)[6]) >> 8 == (turns if tile_order != 1 else 0)
    want = oracle.encode_model_pp(sl, tp, tp_src, src, n_layers, 1, 0, pp_dst)
    for b in range(plan.n_buckets):
        n = R.bucket_check(plan, buckets[b])
        got = {"idx": buckets[b].idx[:n].cpu().numpy(), "val": buckets[b].val[:n].cpu().numpy().view("uint16"),
               "seg_off": buckets[b].seg_off.cpu().numpy()}
        assert_buckets_equal(got, want[b], "bucket %d" % b)
    for i, (o, x) in enumerate(zip(olds, sl)):
        assert (bits(o) == x["new"]).all(), "tensor %d not refreshed" % i
