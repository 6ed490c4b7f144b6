"""Draft calls of several loop-nest classes, interleaved in the segment order: whether a class gets a launch of its own (two classes,
or 2^20 candidates for each of more) or one kernel branches on the class, loading candidates in fours or, in a small population that
is not laid out in fours, one by one, a segment scores as it does in a call of its own."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P  # noqa: F401  (a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CONV, GEMM, DEPTHWISE = w.conv2d(1, 64, 56, 56, 64, 3, 3), w.gemm(512, 512, 512), w.depthwise_conv2d(1, 512, 28, 28, 3, 3)
BATCHED, OTHER = w.batched_gemm(12, 128, 128, 64), w.gemm(128, 768, 3072)


@pytest.mark.parametrize("sgs,lens", [
    ([CONV, GEMM, CONV, OTHER], [300004, 250000, 200008, 400000]),                              # two classes: two launches
    ([DEPTHWISE, GEMM, CONV, OTHER, CONV], [1100000, 600004, 500000, 500000, 600000]),          # three, 2^20 for each: three
    ([DEPTHWISE, GEMM, CONV, OTHER, CONV], [1000000, 600004, 400000, 500000, 600000]),          # three, not 2^20 for each: one
    ([GEMM, BATCHED, OTHER, BATCHED], [500004, 300000, 200000, 100003]),                        # the two kinds of matrix products
    ([CONV, GEMM, CONV, OTHER], [30001, 25000, 0, 4003]), ([GEMM, OTHER], [4001, 300]),
    ([CONV, GEMM], [3, 2]), ([CONV, GEMM, DEPTHWISE], [3001, 2500, 9001]), ([CONV, GEMM, DEPTHWISE], [3004, 2500, 9000]),       # (9001: digits counted)
    ([DEPTHWISE, GEMM, CONV], [200001, 200001, 124285]), ([DEPTHWISE, GEMM, CONV], [200001, 200001, 124286])])   # 2^19 - 1, 2^19
def test_a_segment_scores_as_in_a_call_of_its_own(P, sgs, lens):
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rows = max(w.n_slots(s) for s in sgs)
    tiles = P.random_init(sgs, seg, rows, 17)
    for flags in (P.FUSED_ARITHMETIC, P.REFERENCE_ROUNDING):
        score = P.draft_score(sgs, seg, tiles, flags=flags)
        filtered, idx, _ = P.prior_filter(sgs, seg, tiles, 200, flags=flags) if min(lens) >= 200 else (score, None, None)
        assert torch.equal(filtered.view(torch.int32), score.view(torch.int32))
        if idx is not None:
            assert torch.equal(idx, P.topk(score, seg, 200)[0])
        for t, sg in enumerate(sgs):
            if lens[t] == 0:
                continue
            alone = P.draft_score([sg], [0, lens[t]], tiles[:, seg[t]:seg[t + 1]].contiguous(), flags=flags)
            assert torch.equal(alone.view(torch.int32), score[seg[t]:seg[t + 1]].view(torch.int32)), (t, flags)
