"""Arithmetic payloads by tickets in both forms, of the compacted entries and of every element: bit-identical to the oracle's
over shapes, alignments, tile orders and patterns, and to each other on every pair of patterns.  32-bit word 5 of the
workspace says which form ran (0: of entries, 3: of elements), the buckets' room chooses it."""
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_arith import any_case, check_arith
from test_gpu_parity import T
from test_gpu_unaligned import packed_case

pytestmark = pytest.mark.gpu

TILE = 8192
OF_ENTRIES, OF_ELEMENTS = 0, 3


def form(c):
    return int(c.ws.view(torch.int32)[5])


def shapes(tp):
    return [T(1, 5, R.REPLICATED), T(TILE * 2 // 765 + 40, 765 * tp, R.SPLIT_COLS), T(tp * 3, 2731, R.SPLIT_ROWS), T(300, 7 * tp, R.SPLIT_COLS),
            T(1, 3 * TILE + 9, R.REPLICATED), T(2 * tp, 12283, R.FUSED_ROWS, [tp, tp]), T(301, 192 * tp, R.SPLIT_COLS), T(tp, 0, R.SPLIT_ROWS)]


@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("p,room,want", [(0.02, 0.1, OF_ENTRIES), (0.25, 0.29, OF_ENTRIES), (0.02, 0.5, OF_ELEMENTS), (0.4, 0.45, OF_ELEMENTS),
                                         (1.0, 1.0, OF_ELEMENTS)])
@pytest.mark.parametrize("packed", [False, True])
def test_either_form(packed, p, room, want, order):
    print("case: arithmetic payloads p=%g room=%g order=%d packed=%s" % (p, room, order, packed), flush=True)
    c = packed_case(shapes(2), 2, p, 5, 1, 3) if packed else any_case(shapes(2), 2, p, seed=int(100 * p) + order)
    for b in c.buckets:
        b.capacity = int(room * b.capacity)
    c.plan.set_tile_order(order)
    check_arith(c)
    assert form(c) == want
    check_arith(c)                                     # the density is known now
    assert form(c) == want


@pytest.mark.parametrize("flags,fp32,want", [(R.ENCODE_ARITH | R.ENCODE_REFRESH, False, OF_ENTRIES), (R.ENCODE_ARITH, True, OF_ENTRIES)])
def test_forms_there_is_one_of(flags, fp32, want):
    print("case: arithmetic payloads flags=%d fp32=%s" % (flags, fp32), flush=True)
    c = packed_case(shapes(3), 3, 0.5, 6, 1, 3, fp32)
    c.plan.set_tile_order(1)
    check_arith(c, flags=flags)
    assert form(c) == want


def test_every_pair_in_both_forms():
    """Of elements (whose every pair the oracle checks elsewhere) and, with refresh, of entries: the same buckets."""
    B = 4096
    plan = R.shard_plan([T(B, 65536, R.REPLICATED)], 1)
    plan.set_tile_order(1)
    ws = R.workspace(plan)
    one, two = R.Bucket(B * 65536, 1), R.Bucket(B * 65536, 1)

    def as_bf16(x):
        return (((x + 0x8000) & 0xFFFF) - 0x8000).to(torch.int16)

    new = as_bf16(torch.arange(65536, dtype=torch.int32, device="cuda").repeat(B))
    for o0 in range(0, 65536, B):
        print("case: both forms, old patterns from %04x" % o0, flush=True)
        old = as_bf16(torch.arange(o0, o0 + B, dtype=torch.int32, device="cuda").repeat_interleave(65536))
        old_tab, new_tab = R.ptr_table([old]), R.ptr_table([new])
        R.delta_encode_ex(plan, old_tab, new_tab, R.BF16, R.ENCODE_ARITH, [one], ws)
        n = R.bucket_check(plan, one)
        assert int(ws.view(torch.int32)[5]) == OF_ELEMENTS and n == B * 65535
        R.delta_encode_ex(plan, old_tab, new_tab, R.BF16, R.ENCODE_ARITH | R.ENCODE_REFRESH, [two], ws)
        assert R.bucket_check(plan, two) == n and int(ws.view(torch.int32)[5]) == OF_ENTRIES
        assert torch.equal(one.idx[:n], two.idx[:n]) and torch.equal(one.val[:n], two.val[:n])
