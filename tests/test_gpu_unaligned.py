"""Tensors that start at any element of a flat buffer and runs that are no multiple of 8 elements:
128-bit loads at every alignment, and vectors that straddle the end of a run.  Expected values come
from the oracle, bit for bit."""
import pytest
import torch

import paper_2605_06534_amd as R
from workloads import synth
from gpu_harness import Case, full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import T
from test_gpu_refresh import check_refresh

pytestmark = pytest.mark.gpu

TILE = 8192


def packed_case(ts, tp, p, seed, first_old, first_new, fp32=False):
    """One tensor right behind the other from the given elements of two flat buffers on."""
    olds, news = [], []
    for i, t, o, n in synth.model_pairs(ts, "bernoulli", seed, "cpu", p=p):
        olds.append(o); news.append(n.float() * (1.0 + 2.0 ** -12) if fp32 else n)
    c = Case(ts, tp, olds, news)

    def pack(xs, first):
        flat = torch.zeros(sum(x.numel() for x in xs) + first, dtype=xs[0].dtype, device="cuda")
        out, at = [], first
        for x in xs:
            v = flat[at:at + x.numel()]
            v.copy_(x.reshape(-1))
            out.append(v)
            at += x.numel()
        return out
    c.old, c.new = pack(olds, first_old), pack(news, first_new)
    c.old_tab, c.new_tab = R.ptr_table(c.old), R.ptr_table(c.new)
    return c


def shapes(run, tp):
    # column blocks of `run`, enough rows for several tiles and a ragged end; neighbours of odd sizes around them
    rows = (TILE * 2 + 37) // run + 1
    return [T(1, 5, R.REPLICATED), T(rows, run * tp, R.SPLIT_COLS), T(tp * 3, 2731, R.SPLIT_ROWS), T(1, TILE + 9, R.REPLICATED),
            T(2 * tp, 1023, R.FUSED_ROWS, [tp, tp])]


@pytest.mark.parametrize("run", [7, 8, 9, 15, 16, 71, 513, 765, TILE - 1, TILE + 3])
@pytest.mark.parametrize("fp32", [False, True])
def test_packed_tensors(run, fp32, tile_order):
    print("case: packed run=%d fp32=%s" % (run, fp32), flush=True)
    for tp, first_old, first_new, p in [(2, 1, 3, 0.05), (3, 7, 0, 0.9)]:
        ts = shapes(run, tp)
        full_parity(packed_case(ts, tp, p, run, first_old, first_new, fp32))
        check_arith(packed_case(ts, tp, p, run + 1, first_old, first_new, fp32))
        check_refresh(packed_case(ts, tp, p, run + 2, first_old, first_new, fp32))


def test_packed_tensors_counted_ahead(tile_order):
    """Few workers and dense changes: the count-only pass over tiles whose vectors straddle runs."""
    ts = [T(4096, 765 * 2, R.SPLIT_COLS), T(2048, 1530, R.SPLIT_ROWS)]
    for workers, p in [(66, 0.6), (97, 1.0)]:
        print("case: packed counted ahead workers=%d p=%g" % (workers, p), flush=True)
        c = packed_case(ts, 2, p, workers, 1, 3)
        c.plan.set_worker_cap(workers)
        full_parity(c, check_dense=False)
        w = c.ws.view(torch.int32)
        assert int(w[2]) + int(w[3]) > 0, "the count-only pass never ran"
