"""Tensors that start at any element of a flat buffer and runs that are no multiple of 8 elements:
128-bit loads at every alignment, and vectors that straddle the end of a run.  Expected values come
from the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from workloads import synth
from gpu_harness import Case, bits, full_parity, host_new
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


@pytest.mark.parametrize("run", [1, 7, 8, 9, 16, 71, 513, 765, TILE - 1, TILE + 3])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("first_dst", [0, 1, 4, 7])
def test_dense_copy_between_packed_buffers(run, fp32, first_dst):
    """Source and destination tensors at any element, also from a sender that holds a part of every row."""
    print("case: packed dense run=%d fp32=%s dst at %d" % (run, fp32, first_dst), flush=True)
    for tp, tp_src, first in [(2, 1, 3), (2, 4, 0), (4, 2, 5)]:
        ts = shapes(run, max(tp, tp_src))
        c = packed_case(ts, tp, 0.5, run, 1, first, fp32)
        new = [oracle.rne_bf16(host_new(n)) if fp32 else bits(n) for n in c.new]
        for d in range(tp):
            want, dst = [], []
            for t, x in zip(ts, new):
                want.append(oracle.dense_shard(x, t["rows"], t["cols"], t["rule"], t["sections"], tp, d))
            total = sum(w.size for w in want)
            flat = torch.full((total + first_dst + 16,), 0x5A5A, dtype=torch.int16, device="cuda")
            at = first_dst
            for w in want:
                dst.append(flat[at:at + w.size])
                at += w.size
            for s in range(tp_src):                     # every sender's part, from its own packed slice
                src = []
                for t, x in zip(ts, c.new):
                    m = x.view(t["rows"], t["cols"])
                    src.append(shard(m, t, tp_src, s))
                store = torch.cat([torch.zeros(first, dtype=src[0].dtype, device="cuda")] + [x.reshape(-1) for x in src])
                views, at = [], first
                for x in src:
                    views.append(store[at:at + x.numel()])
                    at += x.numel()
                plan = R.shard_plan(ts, tp, tp_src, s)
                R.dense_copy(plan, d, R.ptr_table(views), c.new_dtype, R.ptr_table(dst))
                torch.cuda.synchronize()
            got = flat.cpu().numpy().view(np.uint16)
            assert np.array_equal(got[first_dst:first_dst + total], np.concatenate(want))
            assert (got[:first_dst] == 0x5A5A).all() and (got[first_dst + total:] == 0x5A5A).all()


def shard(m, t, tp, d):
    """Shard d of a full matrix, by slicing."""
    if t["rule"] == R.SPLIT_ROWS:
        k = m.shape[0] // tp
        return m[d * k:(d + 1) * k]
    if t["rule"] == R.SPLIT_COLS:
        k = m.shape[1] // tp
        return m[:, d * k:(d + 1) * k]
    if t["rule"] == R.FUSED_ROWS:
        out, at = [], 0
        for rows in t["sections"]:
            k = rows // tp
            out.append(m[at + d * k:at + (d + 1) * k])
            at += rows
        return torch.cat(out)
    return m
