"""Populations of several loop-nest classes: one kernel branches over the four classes with closed forms, another over those and the
generic one.  A candidate's score has the same bits from either as from the kernel of its class alone, and the selection behind it
is that of the two calls."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, dev  # noqa: F401  (P is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HW = w.Device(T_p=3.3e12, T_m=4.1e11, m_l0=96, m_l1=20000, pu_l1=3, n_l1=24, pu_l2=7, n_l2=5)
CLOSED = [w.conv2d(1, 64, 56, 56, 64, 3, 3), w.gemm(512, 512, 512), w.depthwise_conv2d(1, 512, 28, 28, 3, 3), w.batched_gemm(12, 128, 128, 64),
          w.gemm(1024, 256, 256, dtype_bytes=2, rd_levels=3, frag=(16, 16, 16))]
GENERIC = w.Subgraph("gemm_bt", 2, 1, (96, 80, 72), 4, 3, 4, (0, 0, 0), (w.Buffer((((0, 1),), ((2, 1),))), w.Buffer((((1, 1),), ((2, 1),)))),
                     w.Buffer((((0, 1),), ((1, 1),))), HW)


@pytest.mark.parametrize("lens", [[1024, 1025, 4, 2000, 1], [140000, 131073, 120001, 90003, 60002], [300001, 290000, 280004, 270008, 300003]])
@pytest.mark.parametrize("generic", [False, True])
def test_a_class_among_others_scores_as_alone(P, lens, generic):
    sgs = CLOSED + ([GENERIC] if generic else [])
    lens = lens + ([777] if generic else [])
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, rows = int(seg[-1]), max(w.n_slots(s) for s in sgs)
    tiles = np.ones((rows, n), np.uint16)
    for t, sg in enumerate(sgs):
        tl, _ = w.sample_population(sg, lens[t], seed=12, stream=t)
        tiles[: tl.shape[0], seg[t]:seg[t + 1]] = tl
    device_tiles = dev(tiles)
    for flags in (P.REFERENCE_ROUNDING, P.FUSED_ARITHMETIC, P.FUSED_ARITHMETIC | P.NO_COMPUTE_PENALTY):
        together = P.draft_score(sgs, seg, device_tiles, flags=flags)
        k = min(*lens, 4096)
        score, idx, val = P.prior_filter(sgs, seg, device_tiles, k, flags=flags)
        want, want_val = P.topk(together, seg, k)
        assert torch.equal(score.view(torch.int32), together.view(torch.int32)) and torch.equal(idx, want) and torch.equal(val, want_val)
        for t, sg in enumerate(sgs):
            alone = P.draft_score([sg], [0, lens[t]], device_tiles[:, int(seg[t]):int(seg[t + 1])].contiguous(), flags=flags)
            assert torch.equal(alone.view(torch.int32), together[int(seg[t]):int(seg[t + 1])].view(torch.int32))


@pytest.mark.parametrize("n_sg", [1, 7, 8, 9, 10, 40])
def test_tables_that_fit_a_launch_and_tables_that_do_not(P, n_sg):
    """different subgraphs, so that every one has a table entry of its own: those of a few travel with the launch itself"""
    sgs = [w.gemm(64 + 32 * t, 128, 256) for t in range(n_sg)]
    seg = np.concatenate([[0], np.cumsum([300 + t for t in range(n_sg)])]).astype(np.int64)
    tiles = P.random_init(sgs, seg, max(w.n_slots(s) for s in sgs), 5)
    score = P.draft_score(sgs, seg, tiles)
    filtered, idx, _ = P.prior_filter(sgs, seg, tiles, 70)
    assert torch.equal(filtered.view(torch.int32), score.view(torch.int32)) and torch.equal(idx, P.topk(score, seg, 70)[0])
    for t, sg in enumerate(sgs):
        alone = P.draft_score([sg], [0, int(seg[t + 1] - seg[t])], tiles[:, int(seg[t]):int(seg[t + 1])].contiguous())
        assert torch.equal(alone.view(torch.int32), score[int(seg[t]):int(seg[t + 1])].view(torch.int32))


@pytest.mark.parametrize("sg", CLOSED + [GENERIC])
@pytest.mark.parametrize("n", [1, 63, 65, 1025, 262144, 262145])
def test_one_candidate_per_thread_and_four(P, sg, n):
    """a class's own kernel at either width: the symbol dump's launch has four to a thread at any size"""
    tiles = P.random_init([sg], [0, n], w.n_slots(sg), 31)
    for flags in (0, P.FUSED_ARITHMETIC, P.REFERENCE_ROUNDING | P.NO_MEMORY_PENALTY):
        score = P.draft_score([sg], [0, n], tiles, flags=flags)
        dumped, _ = P.draft_score([sg], [0, n], tiles, flags=flags, symbols=True)
        assert torch.equal(score.view(torch.int32), dumped.view(torch.int32))
