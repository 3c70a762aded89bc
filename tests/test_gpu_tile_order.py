"""The library's own choice of tile order: from the density that rose_bucket_check read back for
the plan's last launch (timed below 4 %, neighbours below 7.5 %, spread above), whatever the buckets
could hold; the buckets are the oracle's in every case."""
import pytest
import torch

import paper_2605_06534_amd as R
from paper_2605_06534_amd import binding
from workloads import models
from gpu_harness import full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import bern_case
from test_gpu_refresh import check_refresh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,want", [(0.02, binding.TILE_ORDER_TIMED), (0.055, binding.TILE_ORDER_NEIGHBOURS),
                                    (0.12, binding.TILE_ORDER_SPREAD)])
def test_order_follows_the_density_read_back(p, want):
    print("case: auto tile order at p=%g" % p, flush=True)
    ts = models.decoder(2, 512, 8, 8, 64, 1408, 4096, fused=True)
    c = bern_case(ts, 4, p, seed=7)
    caps = [b.capacity for b in c.buckets]
    full = [c.plan.bucket_capacity(d) for d in range(4)]
    assert c.plan.pick_tile_order(full) == binding.TILE_ORDER_SPREAD          # nothing known, nothing bounded
    full_parity(c)                                                             # encodes, checks every bucket, applies
    assert c.plan.pick_tile_order(full) == want
    assert c.plan.pick_tile_order(caps) == want
    full_parity(c)                                                             # the launch in the picked order
    torch.cuda.synchronize()


@pytest.mark.parametrize("p,want", [(0.02, binding.TILE_ORDER_TIMED), (0.045, binding.TILE_ORDER_NEIGHBOURS),
                                    (0.06, binding.TILE_ORDER_NEIGHBOURS), (0.12, binding.TILE_ORDER_SPREAD)])
@pytest.mark.parametrize("arith", [False, True])
def test_launches_in_the_order_picked(p, want, arith):
    """An update too large for reading it twice, in a workspace with no room to park entries: one launch before any
    density is known, one in the order picked from the density read back, one after a wrong guess (a tenth of the
    density).  The workspace's words 4 (tiles of an update without tickets) and 1024 (the ticket counter) show that
    tickets were taken."""
    print("case: launch in the picked order p=%g arith=%s" % (p, arith), flush=True)
    ts = models.decoder(2, 1024, 16, 16, 64, 2816, 4096, fused=True)
    c = bern_case(ts, 4, p, seed=9)
    c.ws = c.ws[:(c.plan.workspace_bytes() - c.plan.n_tiles() * 2016 * 4 + 7) // 8].clone()
    for what in ("unknown", "known", "guessed too low"):
        c.ws.fill_(0)
        for b in c.buckets:
            b.idx.fill_(-7)
        if what == "guessed too low":
            few = R.Bucket(8, len(ts))
            few.capacity = 1 << 40
            few.seg_off[-1] = int(0.1 * p * c.plan.bucket_capacity(0))
            R.bucket_check(c.plan, few)
            assert c.plan.pick_tile_order([b.capacity for b in c.buckets]) == binding.TILE_ORDER_TIMED
        elif what == "known":
            assert c.plan.pick_tile_order([b.capacity for b in c.buckets]) == want
        check_arith(c) if arith else full_parity(c, check_dense=False)
        assert int(c.ws.view(torch.int32)[4]) == 0 and int(c.ws.view(torch.int32)[1024]) > 0, what


@pytest.mark.parametrize("refresh", [False, True])
@pytest.mark.parametrize("fp32,few,more", [(False, 0.06, 0.07), (True, 0.052, 0.062)])
def test_four_neighbours_a_ticket(fp32, few, more, refresh):
    """The neighbours order takes four tiles a ticket where the buckets have room for little more than its line, three where
    they have for more, and three with refresh; the workspace's word 6 says how many a launch took."""
    print("case: neighbours, room for %g and %g, fp32 %d, refresh %d" % (few, more, fp32, refresh), flush=True)
    ts = models.decoder(2, 1024, 16, 16, 64, 2816, 4096, fused=True)
    for room in (few, more):
        c = bern_case(ts, 4, 0.045, seed=11)
        if fp32:
            c.new = [n.float() for n in c.new]
            c.new_tab, c.new_dtype = R.ptr_table(c.new), R.FP32_RNE
        c.plan.set_tile_order(binding.TILE_ORDER_NEIGHBOURS)
        for b in c.buckets:
            b.capacity = int(room * b.capacity)
        c.ws.fill_(-1)
        check_refresh(c) if refresh else full_parity(c, check_dense=False)
        assert int(c.ws.view(torch.int32)[6]) & 255 == (4 if room == few and not refresh else 3), room
