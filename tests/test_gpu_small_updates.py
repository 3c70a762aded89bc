"""Small updates go in two launches instead of tickets: same buckets, refresh and payloads, from empty
tensors up to the largest update of that kind and the smallest one beyond.  Expected values come from
the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import full_parity
from test_gpu_arith import check_arith
from test_gpu_parity import T, bern_case
from test_gpu_refresh import check_refresh
from test_gpu_unaligned import packed_case, shapes

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.mark.parametrize("p", [0.0, 0.03, 1.0])
@pytest.mark.parametrize("numel", [1, 7, 8, 9, TILE - 1, TILE, TILE + 1, 3 * TILE + 17])
def test_flat_sizes(numel, p):
    print("case: small flat numel=%d p=%g" % (numel, p), flush=True)
    ts = [T(1, numel, R.REPLICATED), T(0, 16, R.SPLIT_ROWS), T(2, numel, R.SPLIT_ROWS)]
    full_parity(bern_case(ts, 2, p, seed=numel))
    check_arith(bern_case(ts, 2, p, seed=numel + 1))
    check_refresh(bern_case(ts, 2, p, seed=numel + 2))


@pytest.mark.parametrize("run", [7, 9, 513, 765])
@pytest.mark.parametrize("fp32", [False, True])
def test_packed(run, fp32):
    print("case: small packed run=%d fp32=%s" % (run, fp32), flush=True)
    for tp, first_old, first_new, p in [(2, 1, 3, 0.05), (3, 7, 0, 0.9)]:
        ts = shapes(run, tp)
        full_parity(packed_case(ts, tp, p, run, first_old, first_new, fp32))
        check_arith(packed_case(ts, tp, p, run + 1, first_old, first_new, fp32))
        check_refresh(packed_case(ts, tp, p, run + 2, first_old, first_new, fp32))


@pytest.mark.parametrize("tiles", [2560, 2561, 4096, 4097])
def test_both_sides_of_the_line(tiles):
    print("case: small tiles=%d" % tiles, flush=True)
    full_parity(bern_case([T(1, tiles * TILE, R.REPLICATED)], 1, 0.01, seed=tiles), check_dense=False)


@pytest.mark.parametrize("tiles", [2560, 2561])
def test_refresh_on_both_sides_of_the_line(tiles):
    print("case: small refresh tiles=%d" % tiles, flush=True)
    check_refresh(bern_case([T(tiles, TILE, R.SPLIT_ROWS)], 1, 0.02, seed=tiles))


def test_overflow_is_reported_and_bounded():
    print("case: small overflow", flush=True)
    c = bern_case([T(64, 512, R.SPLIT_ROWS), T(1, 3000, R.REPLICATED)], 2, 0.25, seed=2, capacity=1000)
    want = oracle.encode_model(c.records(), 2)
    for b in c.buckets:                                 # room behind the capacity to watch
        b.idx = torch.full((1064,), -7, dtype=torch.int32, device="cuda")
        b.val = torch.full((1064,), -7, dtype=torch.int16, device="cuda")
    c.encode()
    for d, b in enumerate(c.buckets):
        with pytest.raises(R.RoseError) as e:
            R.bucket_check(c.plan, b)
        assert e.value.required == want[d]["seg_off"][-1] > 1000
        assert np.array_equal(b.seg_off.cpu().numpy(), want[d]["seg_off"])
        assert np.array_equal(b.idx[:1000].cpu().numpy(), want[d]["idx"][:1000])
        assert np.array_equal(b.val[:1000].cpu().numpy().view(np.uint16), want[d]["val"][:1000])
        assert (b.idx[1000:] == -7).all() and (b.val[1000:] == -7).all()


def test_checks_from_many_threads():
    """More bucket checks at a time than a plan has pinned words, each on a stream of its own."""
    import threading
    print("case: threaded checks", flush=True)
    ts = [T(1, 4096, R.REPLICATED)]
    plan = R.shard_plan(ts, 1)
    plan.upload()
    buckets = [R.Bucket(4096, 1) for _ in range(96)]
    for i, b in enumerate(buckets):
        b.seg_off.copy_(torch.tensor([0, i + 1], dtype=torch.int64))
    torch.cuda.synchronize()
    wrong, right = [], [0] * 96

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    if R.bucket_check(plan, buckets[i]) == i + 1:
                        right[i] += 1
        except Exception as e:                          # would only end the thread
            wrong.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(96)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong and right == [20] * 96


def test_two_launches_in_a_graph():
    """The counting and the writing launch captured once and replayed on changed inputs, with eager work between."""
    from gpu_harness import assert_buckets_equal, bits
    from workloads import models
    print("case: small update in a graph", flush=True)
    c = bern_case(models.decoder(2, 320, 8, 8, 40, 1376, 2048, fused=True), 2, 0.05, seed=91)
    c.encode()
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            R.delta_encode(c.plan, c.old_tab, c.new_tab, c.new_dtype, c.buckets, c.ws)
    torch.cuda.synchronize()
    for rep in range(4):
        for n in c.new:
            n.copy_(torch.roll(n, rep))
        for b in c.buckets:
            b.idx.fill_(-7)
            b.seg_off.fill_(-1)
        c.ws.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        want = oracle.encode_model([dict(t, old=bits(o), new=bits(n)) for t, o, n in zip(c.tensors, c.old, c.new)], c.tp)
        for d in range(c.tp):
            assert_buckets_equal(c.host_bucket(d), want[d], "replay %d shard %d" % (rep, d))


def test_diagnostic_words_are_this_launch_s():
    """Words 2 and 3 of the workspace count what happened in the launch (here: no tickets, nothing to count),
    not what the workspace held before."""
    print("case: diagnostic words", flush=True)
    c = bern_case([T(64, 512, R.SPLIT_ROWS), T(1, 3000, R.REPLICATED)], 2, 0.1, seed=3)
    c.ws.fill_(-1)
    c.encode()
    assert c.ws.view(torch.int32)[2:4].tolist() == [0, 0]
