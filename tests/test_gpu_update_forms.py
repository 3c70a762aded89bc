"""How an update of a known density goes, as 32-bit word 5 of its workspace says and as bench.py names its kernels: by tickets
(0), in two launches with its entries parked (1), in two launches that both read the tensors (2)."""
import pytest
import torch

import bench
import paper_2605_06534_amd as R
from paper_2605_06534_amd import binding
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

READ_AGAIN, PARKED, TICKETS = "count_tiles_kernel emit_tiles_kernel", "stage_tiles_kernel emit_staged_kernel", "encode_kernel"


@pytest.mark.parametrize("mib,seen,order,form", [(6, 0.01, 0, READ_AGAIN), (64, 0.01, 0, PARKED), (64, 0.3, 0, READ_AGAIN),
                                                 (64, 0.01, binding.TILE_ORDER_TIMED, TICKETS), (400, 0.2, 0, TICKETS)])
def test_kernels_of_an_update(mib, seen, order, form):
    print("case: form of %d MiB at %g, order %d" % (mib, seen, order), flush=True)
    n = (mib << 20) // 4
    plan = R.shard_plan([T(n // 4096, 4096, R.SPLIT_ROWS)], 1)
    plan.set_tile_order(order)
    weights = torch.zeros(n, dtype=torch.int16, device="cuda")
    tab = R.ptr_table([weights])
    b = R.Bucket(1024, 1)
    b.seg_off[-1], b.capacity = int(seen * n), 1 << 40
    R.bucket_check(plan, b)
    b.capacity = 1024
    ws = R.workspace(plan)
    ws.fill_(-1)
    R.delta_encode(plan, tab, tab, R.BF16, [b], ws)
    assert R.bucket_check(plan, b) == 0
    words = ws.view(torch.int32)
    assert " ".join(k.split("<")[0] for k in bench.encode_kernels(int(words[5]), 0, 0)) == form
    assert int(words[4]) == (0 if form == TICKETS else plan.n_tiles()) and (int(words[1024]) > 0) == (form == TICKETS)


@pytest.mark.parametrize("mib,seen,room,form", [
    (13, None, 1.0, READ_AGAIN), (64, None, 1.0, READ_AGAIN), (90, None, 1.0, TICKETS),         # nothing known
    (16, None, 0.05, PARKED), (16, None, 0.12, READ_AGAIN), (24, None, 0.11, READ_AGAIN), (25, None, 0.11, PARKED), (47, None, 0.13, READ_AGAIN), (48, None, 0.13, PARKED),
    (30, None, 0.02, PARKED), (64, None, 0.3, READ_AGAIN), (200, None, 0.02, PARKED),           # what the buckets hold
    (30, 0.01, 1.0, READ_AGAIN), (30, 0.01, 0.02, PARKED), (30, 0.02, 0.01, PARKED),
    (64, 0.01, 1.0, PARKED), (64, 0.3, 0.02, READ_AGAIN), (280, 0.01, 1.0, PARKED),             # the last density
    (320, 0.01, 1.0, TICKETS), (320, 0.01, 0.02, PARKED), (800, 0.01, 1.0, TICKETS), (800, 0.01, 0.012, PARKED),
    (800, 0.01, 0.1, TICKETS)])
def test_a_wrong_guess(mib, seen, room, form):
    """The form is chosen by a density that may be outdated only where that costs little if it is."""
    print("case: form of %d MiB, seen %s, room for %g" % (mib, seen, room), flush=True)
    n = (mib << 20) // 4
    plan = R.shard_plan([T(n // 4096, 4096, R.SPLIT_ROWS)], 1)
    weights = torch.zeros(n, dtype=torch.int16, device="cuda")
    tab = R.ptr_table([weights])
    b = R.Bucket(int(room * n), 1)
    if seen is not None:
        b.seg_off[-1], b.capacity = int(seen * n), 1 << 40
        R.bucket_check(plan, b)
        b.capacity = int(room * n)
    ws = R.workspace(plan)
    ws.fill_(-1)
    R.delta_encode(plan, tab, tab, R.BF16, [b], ws)
    assert R.bucket_check(plan, b) == 0
    assert " ".join(k.split("<")[0] for k in bench.encode_kernels(int(ws.view(torch.int32)[5]), 0, 0)) == form
