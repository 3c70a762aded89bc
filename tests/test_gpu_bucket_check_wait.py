"""rose_bucket_check reads the total back into a pinned word and waits for the stream: the same answer at once, behind work
that lasts, on other streams, from several threads and for a plan that is resident nowhere."""
import threading

import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


def bucket(total, capacity=1000):
    b = R.Bucket(capacity, 1)
    b.seg_off.copy_(torch.tensor([0, total]))
    return b


@pytest.mark.parametrize("cycles", [0, 20_000, 5_000_000])
@pytest.mark.parametrize("uploaded", [True, False])
def test_totals(cycles, uploaded):
    print("case: bucket check behind %d cycles, uploaded=%s" % (cycles, uploaded), flush=True)
    plan = R.shard_plan([T(64, 64, R.SPLIT_ROWS)], 1)
    if uploaded:
        plan.upload()
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            b = bucket(0)
            for total in (1, 1000, 0, 777):
                later = torch.tensor([0, total], device="cuda")
                if cycles:
                    torch.cuda._sleep(cycles)
                b.seg_off.copy_(later)
                assert R.bucket_check(plan, b) == total
            b.seg_off[1] = 1001
            with pytest.raises(R.RoseError) as e:
                R.bucket_check(plan, b)
            assert e.value.required == 1001
            b.seg_off[1] = -1
            with pytest.raises(R.RoseError):
                R.bucket_check(plan, b)
        torch.cuda.synchronize()


def test_threads():
    print("case: bucket checks from eight threads", flush=True)
    plan = R.shard_plan([T(64, 64, R.SPLIT_ROWS)], 1)
    plan.upload()
    buckets = [[bucket(100 * i + j) for j in range(20)] for i in range(8)]
    torch.cuda.synchronize()
    got = [None] * 8

    def check(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[i] = [R.bucket_check(plan, b) for _ in range(10) for b in buckets[i]]

    threads = [threading.Thread(target=check, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [[100 * i + j for _ in range(10) for j in range(20)] for i in range(8)]
