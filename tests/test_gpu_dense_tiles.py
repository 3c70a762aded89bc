"""Dense copies of pieces around whole tiles, to destinations that begin anywhere: byte-identical to the oracle's slices, and
nothing around them is written.  A copy has no tile for a piece to be moved by, so its numbering of tiles is its own."""
import numpy as np
import pytest
import torch

import paper_2605_06534_amd as R
from oracle import oracle
from gpu_harness import host_new
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

TILE, LINE = 8192, 64
LENS = [1, 7, TILE - 1, TILE, TILE + 1, 2 * TILE - LINE + 1, 2 * TILE - LINE + 2, 2 * TILE - 1, 2 * TILE, 2 * TILE + 9, 5 * TILE - 3]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("at", [0, 1, 8, LINE - 1])
@pytest.mark.parametrize("tp", [1, 3])
def test_whole_tiles(tp, at, fp32):
    print("case: dense copy of whole tiles, tp=%d, %d elements behind a line, fp32=%s" % (tp, at, fp32), flush=True)
    ts = [T(tp, n, R.SPLIT_ROWS) for n in LENS] + [T(1, 2 * TILE, R.REPLICATED), T(0, 5, R.REPLICATED),
                                                  T(64, 192 * tp, R.SPLIT_COLS), T(2 * tp, TILE, R.FUSED_ROWS, [tp, tp])]
    g = torch.Generator().manual_seed(tp)
    new = [torch.randint(-2 ** 31, 2 ** 31 - 1, (t["rows"] * t["cols"],), generator=g, dtype=torch.int32).view(torch.float32).cuda() if fp32
           else torch.randint(-2 ** 15, 2 ** 15 - 1, (t["rows"] * t["cols"],), generator=g, dtype=torch.int16).view(torch.bfloat16).cuda()
           for t in ts]
    plan = R.shard_plan(ts, tp)
    tab = R.ptr_table(new)
    for d in range(tp):
        spots, o = [], 0
        for t in range(len(ts)):
            o = -(-o // LINE) * LINE + at
            spots.append((o, plan.local_numel(t, d)))
            o += spots[-1][1] + 1
        flat = torch.full((o + LINE,), 0x5A5A, dtype=torch.int16, device="cuda")
        R.dense_copy(plan, d, tab, R.FP32_RNE if fp32 else R.BF16, R.ptr_table([flat[a:a + max(n, 1)] for a, n in spots]))
        want = np.full(o + LINE, 0x5A5A, dtype=np.uint16)
        for (a, n), t, w in zip(spots, ts, new):
            bits = host_new(w)
            bits = oracle.rne_bf16(bits) if fp32 else bits
            if n:
                want[a:a + n] = oracle.dense_shard(bits, t["rows"], t["cols"], t["rule"], t["sections"], tp, d)
        assert np.array_equal(flat.cpu().numpy().view(np.uint16), want), "shard %d" % d
