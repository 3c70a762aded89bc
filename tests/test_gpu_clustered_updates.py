"""Updates that go in two launches and whose changes lie close together, so that neighbouring tiles hold more than their
slots: correct, and not slower than their reading takes (a fine-tuned part of an otherwise frozen model)."""
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T
from test_gpu_staged_updates import CHECKS, PARKED, form, know_density, make, tiles_without_tickets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", sorted(CHECKS))
@pytest.mark.parametrize("mib,tp,p,dense,fp32", [(14, 1, 0.001, 20, False), (60, 2, 0.002, 70, True), (70, 4, 0.002, 300, False),
                                                 (290, 2, 0.001, 900, False)])
def test_runs_of_dense_tiles(mib, tp, p, dense, fp32, what):
    print("case: %d dense tiles in %d MiB tp=%d %s fp32=%s" % (dense, mib, tp, what, fp32), flush=True)
    c = make(mib, tp, 513, p, mib + dense, fp32, dense)
    know_density(c)
    CHECKS[what](c)
    assert tiles_without_tickets(c) == c.plan.n_tiles() and form(c) == PARKED


@pytest.mark.parametrize("what", sorted(CHECKS))
@pytest.mark.parametrize("entries", [256, 300, 2016])
def test_small_slots(entries, what):
    """Room for so many entries a tile, tiles that hold nearly as many or 8192."""
    print("case: slots of %d entries, %s" % (entries, what), flush=True)
    c = make(50, 2, 8, 0.16 if entries == 2016 else 0.006, entries, dense=2)
    base = c.plan.workspace_bytes() - c.plan.n_tiles() * 2016 * 4
    c.ws = torch.full(((base + c.plan.n_tiles() * entries * 4) // 8 + 1,), -1, dtype=torch.int64, device="cuda")
    CHECKS[what](c)
    assert form(c) == PARKED


def test_time_of_changes_that_lie_together():
    """2 % of 192 MiB: evenly spread, and all of them in neighbouring tiles (1.14 times as long where every such tile has
    a workgroup of its own, 3.1 where 8 go one behind the other)."""
    n = 192 << 18
    rows = n // 4096
    plan = R.shard_plan([T(rows, 4096, R.SPLIT_ROWS)], 1)
    plan.upload()
    old = torch.randint(-30000, 30000, (n,), dtype=torch.int16, device="cuda")
    spread, together = old.clone(), old.clone()
    spread[::50] ^= 1
    together[:n // 50] ^= 1
    ws, b = R.workspace(plan), R.Bucket(n, 1)
    old_tab = R.ptr_table([old])
    us = {}
    for what, new in (("spread", spread), ("together", together)):
        tab = R.ptr_table([new])
        times = []
        for i in range(12):
            R.delta_encode(plan, old_tab, tab, R.BF16, [b], ws)
            assert abs(R.bucket_check(plan, b) - n / 50) <= 1
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(5):
                R.delta_encode(plan, old_tab, tab, R.BF16, [b], ws)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end) * 200)
        us[what] = sorted(times)[len(times) // 2]
        assert int(ws.view(torch.int32)[4]) == plan.n_tiles()
    print("case: changes spread %.1f us, together %.1f us" % (us["spread"], us["together"]), flush=True)
    assert us["together"] < 2 * us["spread"], us
