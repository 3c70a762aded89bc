"""Pieces of several tiles whose tensors begin anywhere: their tiles are moved down to lines of the old tensor,
the vectors at the piece's ends to its first and last eight elements.  Every form of the launch is compared, byte for byte,
with the same update whose tensors begin at lines (which the oracle checks), over lengths around whole tiles."""
import pytest
import torch

import paper_2605_06534_amd as R
from gpu_harness import full_parity
from test_gpu_parity import T
from test_gpu_unaligned import packed_case

TILE, LINE = 8192, 64
LENS = [TILE, TILE + 1, TILE + LINE - 1, 2 * TILE - LINE + 1, 2 * TILE - LINE + 2, 2 * TILE - 1, 2 * TILE, 2 * TILE + 7, 3 * TILE + 5]
MOVED = [4 * TILE - LINE + 1, 4 * TILE + 1, 5 * TILE + 7, 6 * TILE - LINE, 6 * TILE + LINE - 1, 7 * TILE - LINE + 1]


def tensors(tp, mib):
    ts = [T(tp, n, R.SPLIT_ROWS) for n in LENS + MOVED] + [T(1, 3 * TILE, R.REPLICATED), T(2 * tp, 2 * TILE + 9, R.FUSED_ROWS, [tp, tp]),
                                                  T(TILE // 8 + 3, 24 * tp, R.SPLIT_COLS), T(301, 192 * tp, R.SPLIT_COLS),
                                                  T(tp, 32 * TILE, R.SPLIT_ROWS), T(33 * TILE // 192, 192 * tp, R.SPLIT_COLS)]
    return ts + [T(tp * 2, (mib << 20) // 4 // tp // 2, R.SPLIT_ROWS)] if mib else ts


def test_tiles_of_a_plan():
    for n, tiles in zip(LENS + [31 * TILE, 32 * TILE - LINE + 1, 32 * TILE - LINE + 2, 32 * TILE], [1, 2, 2, 2, 3, 3, 3, 3, 4, 32, 32, 33, 33]):
        assert R.shard_plan([T(1, n, R.SPLIT_ROWS)], 1).n_tiles() == tiles, n
    assert R.shard_plan([T(TILE, 4, R.SPLIT_COLS)], 2).n_tiles() == 4          # rows of no whole lines: not moved
    assert R.shard_plan([T(TILE, 128, R.SPLIT_COLS)], 2).n_tiles() == 2 * (64 + 1)
    assert R.shard_plan([T(1, (1 << 31) - 8, R.REPLICATED)], 1).n_tiles() == 1 << 18


def run(plan, olds, news, at_old, at_new, flags, order):
    """Each tensor `at` elements behind a line of its flat buffer."""
    def place(xs, at):
        flat, views, o = torch.zeros(sum(x.numel() + 4 * LINE for x in xs), dtype=xs[0].dtype, device="cuda"), [], 0
        for x in xs:
            o = -(-o // LINE) * LINE + at
            views.append(flat[o:o + x.numel()])
            views[-1].copy_(x.reshape(-1))
            o += x.numel()
        return flat, views
    (keep_o, old), (keep_n, new) = place(olds, at_old), place(news, at_new)
    buckets = [R.Bucket(plan.bucket_capacity(d), len(olds)) for d in range(plan.n_buckets)]
    for b in buckets:
        b.idx.fill_(-7)
        b.val.fill_(-7)
    plan.set_tile_order(order)
    ws = R.workspace(plan)
    ws.fill_(-1)
    dtype = R.FP32_RNE if new[0].dtype == torch.float32 else R.BF16
    R.delta_encode_ex(plan, R.ptr_table(old), R.ptr_table(new), dtype, flags, buckets, ws)
    torch.cuda.synchronize()
    return [(b.idx, b.val, b.seg_off) for b in buckets], [o.view(torch.int16).clone() for o in old]


@pytest.mark.gpu
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("mib,order", [(0, 0), (16, 0), (0, 1), (16, 2), (16, 3)])
def test_wherever_the_tensors_begin(mib, order, fp32):
    """mib, order: read again, staged, and the tile orders of the ticket kernel."""
    for p in (0.04, 0.9):
        c = packed_case(tensors(3, mib), 3, p, 5, 0, 0, fp32)
        full_parity(c, check_dense=False)
        plans = [(c.plan, c.old, c.new)]
        cols = [T(2500, 4 * 36, R.SPLIT_COLS)]          # a sender's columns: contiguous there, in runs at the receiver
        plans.append((R.shard_plan(cols, 1, 4, 1), [c.old[-1][:2500 * 36]], [c.new[-1][:2500 * 36]]) if mib else plans[0])
        for plan, olds, news in plans:
            for flags in (0, R.ENCODE_ARITH, R.ENCODE_REFRESH, R.ENCODE_ARITH | R.ENCODE_REFRESH):
                want = run(plan, olds, news, 0, 0, flags, order)
                if flags & R.ENCODE_REFRESH:
                    assert all(torch.equal(o.view(-1), n.to(torch.bfloat16).view(torch.int16).view(-1)) for o, n in zip(want[1], news))
                for at_old, at_new in [(1, 1), (LINE - 1, LINE - 1), (8, 8), (7, 40), (33, 0)]:
                    print("case: shifted %d MiB order=%d fp32=%s p=%g flags=%d at %d / %d" % (mib, order, fp32, p, flags, at_old, at_new), flush=True)
                    got = run(plan, olds, news, at_old, at_new, flags, order)
                    for d, (g, w) in enumerate(zip(got[0], want[0])):
                        assert all(torch.equal(x, y) for x, y in zip(g, w)), "bucket %d" % d
                    assert all(torch.equal(x, y) for x, y in zip(got[1], want[1])), "old tensors"
