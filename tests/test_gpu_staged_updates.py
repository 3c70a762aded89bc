"""Updates that go in two launches with their entries parked in slots of the workspace: slots that are too small for
some tiles or for all, groups of tiles that end with a chain, odd widths and alignments, every payload and input type,
and the lines up to which this form is taken.  Expected values come from the oracle, bit for bit; the workspace's 32-bit
words 4 (the tiles of a launch without tickets, else 0) and 5 (1: entries parked, 2: all read again) say which form ran."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import assert_buckets_equal, full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import T, bern_case
from test_gpu_refresh import check_refresh
from test_gpu_unaligned import packed_case

pytestmark = pytest.mark.gpu

TILE = 8192
CHECKS = {"new": lambda c: full_parity(c, check_dense=False), "arith": check_arith, "refresh": check_refresh}


def tensors(mib, tp, run, fp32):
    """Chains that end inside a group of tiles, tiny tensors, column blocks of `run`, and a large tensor up to `mib` read."""
    rows = (TILE * 9 + 37) // run + 1
    ts = [T(1, 5, R.REPLICATED), T(rows, run * tp, R.SPLIT_COLS), T(tp * 3, 2731, R.SPLIT_ROWS), T(1, TILE + 9, R.REPLICATED),
          T(2 * tp, 1023, R.FUSED_ROWS, [tp, tp])]
    left = (mib << 20) // (6 if fp32 else 4) - sum(t["rows"] * t["cols"] for t in ts)
    return ts + [T(max(1, left // (tp * 4096)) * tp, 4096, R.SPLIT_ROWS)]


def make(mib, tp, run, p, seed, fp32=False, dense=0):
    """dense: so many tiles' worth of neighbouring elements of the large tensor all change.  The buckets have room for
    little more than comes: the form goes by that where the density is not known, or not taken."""
    c = packed_case(tensors(mib, tp, run, fp32), tp, p, seed, 1, 3, fp32)
    for b in c.buckets:
        b.capacity = min(b.capacity, int(1.05 * p * b.capacity) + (dense + 2) * TILE)
    if dense:
        part = slice(TILE * 5 + 100, TILE * (5 + dense) + 100)
        was = c.old[-1][part].view(torch.int16)
        c.new[-1][part] = (was ^ 1).view(torch.bfloat16).to(c.new[-1].dtype)
    return c


def know_density(c):
    c.encode()
    counts = []
    for b in c.buckets:
        counts.append(R.bucket_check(c.plan, b))
        b.idx.fill_(-7)
        b.seg_off.fill_(-7)
    c.ws.fill_(-1)
    return counts


def tiles_without_tickets(c):
    return int(c.ws.view(torch.int32)[4])


PARKED, READ_AGAIN = 1, 2


def form(c):
    return int(c.ws.view(torch.int32)[5])


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("what", sorted(CHECKS))
@pytest.mark.parametrize("run,tp,p,dense", [(765, 3, 0.01, 0), (8, 2, 0.2, 0), (7, 1, 0.05, 33)])
def test_small(run, tp, p, dense, what, fp32):
    print("case: staged 13 MiB run=%d tp=%d p=%g %s fp32=%s" % (run, tp, p, what, fp32), flush=True)
    c = make(13, tp, run, p, run, fp32, dense)
    CHECKS[what](c)
    assert tiles_without_tickets(c) == c.plan.n_tiles()
    assert form(c) == (PARKED if p == 0.01 else READ_AGAIN)


@pytest.mark.parametrize("mib,tp,p,what,fp32", [(34, 5, 0.04, "new", False), (81, 2, 0.01, "arith", False), (100, 8, 0.06, "new", True),
                                                (110, 2, 0.1, "refresh", False), (200, 4, 0.02, "refresh", True),
                                                (200, 1, 0.05, "arith", False), (400, 8, 0.004, "new", False),
                                                (400, 2, 0.05, "arith", True)])
def test_groups_of_tiles(mib, tp, p, what, fp32):
    """With the density known, one size for each size of a group; some tiles past their slots."""
    print("case: staged %d MiB tp=%d p=%g %s fp32=%s" % (mib, tp, p, what, fp32), flush=True)
    c = make(mib, tp, 513, p, mib + tp, fp32, dense=21)
    for b, n in zip(c.buckets, know_density(c)):
        b.capacity = n
    CHECKS[what](c)
    assert tiles_without_tickets(c) == c.plan.n_tiles()
    assert form(c) == PARKED


@pytest.mark.parametrize("entries", [0, 31, 255, 256, 300, 2016])
def test_room_for_slots(entries):
    """A workspace with room for so many entries a tile: below 256 nothing is parked."""
    print("case: staged, room for %d" % entries, flush=True)
    c = make(20, 2, 765, 0.06, entries)
    base = c.plan.workspace_bytes() - c.plan.n_tiles() * 2016 * 4
    c.ws = torch.full(((base + c.plan.n_tiles() * entries * 4) // 8 + 1 + 512,), -1, dtype=torch.int64, device="cuda")
    given, c.ws = c.ws, c.ws[:-512]
    full_parity(c, check_dense=False)
    check_arith(c)
    assert (given[-512:] == -1).all()


def test_a_denser_update_than_the_last():
    """The slots were chosen for 1 %, 60 % come."""
    print("case: staged, density misjudged", flush=True)
    ts = tensors(90, 4, 765, False)
    c = bern_case(ts, 4, 0.01, seed=3)
    know_density(c)
    c.new = [n.cuda() for n in bern_case(ts, 4, 0.6, seed=4).new]
    c.old = [o.cuda() for o in bern_case(ts, 4, 0.6, seed=4).old]
    c.old_tab, c.new_tab = R.ptr_table(c.old), R.ptr_table(c.new)
    full_parity(c, check_dense=False)
    assert tiles_without_tickets(c) == c.plan.n_tiles()


@pytest.mark.parametrize("flags", [0, R.ENCODE_ARITH])
def test_overflow(flags):
    """Buckets of half of what comes: nothing behind the capacity is written."""
    print("case: staged overflow flags=%d" % flags, flush=True)
    c = make(30, 2, 765, 0.05, 9, dense=9)
    want = oracle.encode_model(c.records(), 2)
    caps = [int(w["seg_off"][-1]) // 2 + 3 for w in want]
    for b, cap in zip(c.buckets, caps):
        b.capacity = cap
        b.idx.fill_(-7)
        b.val.fill_(-7)
    R.delta_encode_ex(c.plan, c.old_tab, c.new_tab, R.BF16, flags, c.buckets, c.ws)
    torch.cuda.synchronize()
    for d, (b, cap) in enumerate(zip(c.buckets, caps)):
        with pytest.raises(R.RoseError) as e:
            R.bucket_check(c.plan, b)
        assert e.value.required == want[d]["seg_off"][-1]
        assert np.array_equal(b.seg_off.cpu().numpy(), want[d]["seg_off"])
        assert np.array_equal(b.idx[:cap].cpu().numpy() & 0x7FFFFFFF, want[d]["idx"][:cap])
        assert (b.idx[cap:] == -7).all() and (b.val[cap:] == -7).all()


def test_built_in_scratch():
    print("case: staged in the built-in scratch", flush=True)
    c = make(120, 2, 765, 0.03, 17)
    know_density(c)
    R.delta_encode_static(c.plan, c.old_tab, c.new_tab, R.BF16, 0, c.buckets)
    torch.cuda.synchronize()
    want = oracle.encode_model(c.records(), 2)
    for d in range(2):
        assert_buckets_equal(c.host_bucket(d), want[d], "shard %d" % d)


@pytest.mark.parametrize("mib,seen,staged", [(190, 0.11, True), (302, 0.11, False), (430, 0.05, True), (482, 0.05, False)])
def test_lines(mib, seen, staged):
    """Up to which size a density goes without tickets, as the launch itself shows."""
    print("case: staged or not, %d MiB at %g" % (mib, seen), flush=True)
    n = (mib << 20) // 4 // 4096 // 2 * 2
    plan = R.shard_plan([T(n, 4096, R.SPLIT_ROWS)], 1)
    old = torch.zeros(n * 4096, dtype=torch.int16, device="cuda")
    tab = R.ptr_table([old])
    b = R.Bucket(1024, 1)
    b.seg_off[-1] = int(seen * n * 4096)
    b.capacity = 1 << 40
    R.bucket_check(plan, b)
    b.capacity = 1024
    ws = R.workspace(plan)
    ws.fill_(-1)
    R.delta_encode(plan, tab, tab, R.BF16, [b], ws)
    assert R.bucket_check(plan, b) == 0
    assert int(ws.view(torch.int32)[4]) == (plan.n_tiles() if staged else 0)


@pytest.mark.parametrize("what", ["arith", "refresh"])
@pytest.mark.parametrize("run,tp,p", [(765, 3, 0.02), (7, 2, 0.5), (8, 1, 1.0)])
def test_read_again(run, tp, p, what):
    """Below the smallest staged update: every tile is read twice, payloads are formed of all elements."""
    print("case: read again run=%d tp=%d p=%g %s" % (run, tp, p, what), flush=True)
    c = make(6, tp, run, p, run + 1)
    CHECKS[what](c)
    assert tiles_without_tickets(c) == c.plan.n_tiles()
