"""Small updates go in two launches unless a tile order is set; every real model goes by tickets.  What the other
tests check of overflow, refresh, payloads and senders' shares on models of that size is checked here by the
ticket kernels too, in every tile order."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
import test_gpu_arith as arith
import test_gpu_parity as parity
import test_gpu_pipeline as pipeline
import test_gpu_refresh as refresh
import test_gpu_src_sharding as senders
from oracle import oracle
from workloads import models

pytestmark = pytest.mark.gpu

BODIES = {
    "overflow": parity.test_capacity_overflow_is_reported_and_bounded,
    "fp32 special values": parity.test_fp32_rounding_special_values,
    "fp32 masters": parity.test_fp32_master_input,
    "odd shapes": parity.test_odd_shapes_take_the_element_path,
    "odd addresses": parity.test_misaligned_tensors_still_exact,
    "refresh, odd shapes and addresses": refresh.test_refresh_odd_shapes_and_misaligned,
    "refresh, fp32 masters": refresh.test_refresh_fp32_master,
    "refresh, sender's share": refresh.test_refresh_on_a_sender_side_plan,
    "refresh, pipeline stages": pipeline.test_pipeline_sender_refresh_touches_only_its_stage,
    "arithmetic, refresh": lambda: arith.test_arith_with_refresh(False),
    "arithmetic, refresh, fp32 masters": lambda: arith.test_arith_with_refresh(True),
    "arithmetic, fp32 masters": arith.test_arith_fp32_master,
    "arithmetic, odd shapes and addresses": arith.test_arith_odd_shapes_full_tiles_and_misaligned,
    "arithmetic, sender's share": arith.test_arith_sender_side_sharding,
    "sender's share": senders.test_unfused_gqa_and_reverse_sender_order,
}


@pytest.mark.parametrize("name", sorted(BODIES))
def test_by_tickets(name, tile_order):
    print("case: by tickets, %s, order %d" % (name, tile_order), flush=True)
    BODIES[name]()


@pytest.mark.parametrize("flags", [0, R.ENCODE_ARITH])
@pytest.mark.parametrize("p", [0.1, 0.9])
def test_overflow_of_a_large_update(p, flags, tile_order):
    """Buckets of half of what comes, many workgroups, entries copied out of the ring in runs: nothing behind the
    capacity is written, what lies before it and the counts are the oracle's."""
    print("case: overflow by tickets p=%g flags=%d order=%d" % (p, flags, tile_order), flush=True)
    ts = models.decoder(2, 1024, 16, 16, 64, 2816, 4096, fused=True)
    c = parity.bern_case(ts, 2, p, seed=5, capacity=16)
    recs = c.records()
    want = oracle.encode_model(recs, 2)
    if flags:
        want = [oracle.arith_bucket(w, arith.shard_of(c, [r["old"] for r in recs], d)) for d, w in enumerate(want)]
    guard, caps = 4096, [int(w["seg_off"][-1]) // 2 + 3 for w in want]
    for b, cap in zip(c.buckets, caps):
        b.capacity = cap
        b.idx = torch.full((cap + guard,), -7, dtype=torch.int32, device="cuda")
        b.val = torch.full((cap + guard,), -7, dtype=torch.int16, device="cuda")
    R.delta_encode_ex(c.plan, c.old_tab, c.new_tab, R.BF16, flags, c.buckets, c.ws)
    torch.cuda.synchronize()
    for d, (b, cap) in enumerate(zip(c.buckets, caps)):
        with pytest.raises(R.RoseError) as e:
            R.bucket_check(c.plan, b)
        assert e.value.required == want[d]["seg_off"][-1]
        assert np.array_equal(b.seg_off.cpu().numpy(), want[d]["seg_off"])
        assert np.array_equal(b.idx[:cap].cpu().numpy(), want[d]["idx"][:cap])
        assert np.array_equal(b.val[:cap].cpu().numpy().view(np.uint16), want[d]["val"][:cap])
        assert (b.idx[cap:] == -7).all() and (b.val[cap:] == -7).all()
