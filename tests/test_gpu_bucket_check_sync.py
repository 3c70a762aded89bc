"""rose_bucket_check synchronises the stream: once it has returned, the runtime knows all work in front of it to be done
and holds nothing of the call itself back, however short or long that work was."""
import pytest
import torch

import paper_2605_06534_amd as R
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cycles", [0, 2_000, 1_000_000])
def test_the_stream_is_done(cycles):
    print("case: stream after a bucket check behind %d cycles" % cycles, flush=True)
    plan = R.shard_plan([T(64, 64, R.SPLIT_ROWS)], 1)
    plan.upload()
    b = R.Bucket(1000, 1)
    b.seg_off.copy_(torch.tensor([0, 7]))
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            torch.cuda.synchronize()
            done = []
            for _ in range(20):
                if cycles:
                    torch.cuda._sleep(cycles)
                assert R.bucket_check(plan, b) == 7
                done.append(stream.query())
            assert all(done), done
