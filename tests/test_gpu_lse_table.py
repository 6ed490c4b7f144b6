"""pruner_lse on segments with many times more children than S_spec can have different ones, whose scores are looked up in a table of all
of these: subgraphs of one, two and three distinct primes (one, two and four entries per move) and of four (no table), two and three
reduction levels, fragments, segments with and without a table in one call, and populations whose factors have more primes than the
extents say (the table is then not used).  Against the oracle's loop, every integer and every bit of the scores."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as w
from test_gpu_parity import P, dev, check_lse_against_oracle, lse_population  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

ONE = w.gemm(64, 64, 64, dtype_bytes=2, hw=w.toy_device(), rd_levels=3, frag=(16, 16, 16))
TWO = w.gemm(96, 80, 72, hw=w.toy_device())
THREE = w.gemm(60, 90, 64, hw=w.toy_device())
FOUR = w.gemm(210, 64, 32, hw=w.toy_device())
CONV = w.conv2d(1, 8, 12, 12, 16, 3, 3)
DEPTHWISE = w.depthwise_conv2d(1, 32, 28, 28, 3, 3)
BATCHED = w.batched_gemm(4, 32, 48, 40)


@pytest.mark.parametrize("sg", [ONE, TWO, THREE, FOUR, CONV, DEPTHWISE, BATCHED], ids=lambda s: s.name)
@pytest.mark.parametrize("k,n,q16", [(1, 32769, 65536), (17, 40004, 52429), (17, 262144, 52429), (1, 262145, 65536), (17, 262148, 52429), (130, 300003, 30000)])   # (up to 2^18 children are made one to a thread)
def test_one_segment(P, sg, k, n, q16):
    seg, tiles = lse_population([sg], [n], seed=k)
    check_lse_against_oracle(P, [sg], seg, tiles, k, 4, 3 + k, q16)


@pytest.mark.parametrize("n", [60000, 262000])
def test_segments_with_and_without_a_table(P, n):
    sgs = [TWO, CONV, FOUR, BATCHED, ONE]
    seg, tiles = lse_population(sgs, [n, 300, 40001, 700, 33000], seed=4)
    check_lse_against_oracle(P, sgs[:2], seg[:3], np.ascontiguousarray(tiles[:, :seg[2]]), 40, 3, 5, 52000)
    check_lse_against_oracle(P, sgs, seg, tiles, 40, 3, 5, 52000)   # five classes below 2^20: children by a launch of their own


def test_classes_in_launches_of_their_own(P):
    sgs = [TWO, CONV, DEPTHWISE, BATCHED]
    seg, tiles = lse_population(sgs, [400000, 300000, 340002, 9000], seed=6)
    check_lse_against_oracle(P, sgs, seg, tiles, 100, 3, 9, 52429)


@pytest.mark.parametrize("lens", [[60000, 50000, 40000, 33000], [60001, 50002, 40003, 33001]])
def test_several_classes_that_all_have_a_table(P, lens):
    """below 2^20: looked up in one launch, laid out in fours and not"""
    sgs = [TWO, CONV, DEPTHWISE, BATCHED]
    seg, tiles = lse_population(sgs, lens, seed=7)
    check_lse_against_oracle(P, sgs, seg, tiles, 20, 4, 9, 52429)


def test_two_classes_in_one_launch_of_looking_up(P):
    """above 2^18: four to a thread; the first subgraph's primes are more than its extents', so that its children are made there"""
    wide = w.gemm(128, 128, 64, hw=w.toy_device())
    results = []
    for others, more in (([DEPTHWISE], [300000]), ([DEPTHWISE, FOUR, CONV], [300000, 300, 300])):
        sgs = [THREE] + others
        seg, tiles = lse_population(sgs, [40000] + more, seed=8)
        pop = dev(tiles)
        score, spec_t, spec_s, spec_n = P.lse([wide] + others, seg, pop, 64, 3, 2, 52429, flags=P.REFERENCE_ROUNDING)
        rows = min(w.n_slots(s) for s in (wide, DEPTHWISE))
        results.append([pop[:rows, :340000].cpu().numpy(), score[:340000].cpu().numpy(), spec_t[:rows, :128].cpu().numpy(), spec_s[:2].cpu().numpy(), spec_n[:2].cpu().numpy()])
    for alone, beside in zip(*results):
        assert np.array_equal(np.ascontiguousarray(alone).view(np.uint8), np.ascontiguousarray(beside).view(np.uint8))


@pytest.mark.parametrize("n", [40000, 270000])
def test_more_primes_than_the_extents_have(P, n):
    """tiles of 60 x 90 x 64 under a subgraph of powers of two that is large enough for them: the same as in a call of three classes, which
    makes its children by a launch of their own (the oracle refuses such tiles)"""
    wide = w.gemm(128, 128, 64, hw=w.toy_device())
    results = []
    for others in ([], [CONV, BATCHED]):
        sgs = [THREE] + others
        seg, tiles = lse_population(sgs, [n] + [300] * len(others), seed=8)
        pop = dev(tiles)
        score, spec_t, spec_s, spec_n = P.lse([wide] + others, seg, pop, 64, 3, 2, 52429, flags=P.REFERENCE_ROUNDING)
        rows = w.n_slots(wide)
        results.append([pop[:rows, :n].cpu().numpy(), score[:n].cpu().numpy(), spec_t[:rows, :64].cpu().numpy(), spec_s[0].cpu().numpy(),
                        spec_n[:1].cpu().numpy()])
    for alone, beside in zip(*results):
        assert np.array_equal(alone.view(np.uint8), beside.view(np.uint8))


@pytest.mark.parametrize("sgs,lens", [([TWO], [300004]), ([TWO], [8000]), ([TWO, CONV], [1 << 20, 40000])], ids=["table", "made", "classes"])
def test_timing_hook_brackets_a_launch_that_reads(P, sgs, lens):
    """four steps of which the first one alone reads its candidates: the events stand around a launch of that step, results unchanged"""
    seg, tiles = lse_population(sgs, lens, seed=12)
    begin, e0, e1, end = (torch.cuda.Event(enable_timing=True) for _ in range(4))
    for e in (begin, e0, e1, end):
        e.record()
    plain = P.lse(sgs, seg, dev(tiles), 17, 4, 3, 52429)
    pop = dev(tiles)
    got = ctypes.c_int64(-1)
    P.time_dominant_draft_launch(e0, e1, got)
    try:
        begin.record()
        timed = P.lse(sgs, seg, pop, 17, 4, 3, 52429)
        end.record()
        torch.cuda.synchronize()
    finally:
        P.time_dominant_draft_launch(None, None)
    assert got.value == lens[0] * (2 * w.n_slots(sgs[0]) + 4)
    assert 0.0 < e0.elapsed_time(e1) < 50.0
    assert begin.elapsed_time(e0) < e1.elapsed_time(end)
    for a, b in zip(plain, timed):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


FRAGMENT = w.gemm(512, 512, 512, dtype_bytes=2, rd_levels=3, frag=(16, 16, 16))


@pytest.mark.parametrize("flags", ["0", "FUSED_ARITHMETIC", "NO_COMPUTE_PENALTY", "NO_MEMORY_PENALTY", "NO_COMPUTE_PENALTY|FUSED_ARITHMETIC"])
@pytest.mark.parametrize("sgs,lens", [([FRAGMENT], [1 << 20]), ([TWO, DEPTHWISE], [1 << 20, 300004]), ([TWO, CONV, BATCHED], [700000, 300000, 60000])],
                         ids=["one", "two", "three"])
def test_scores_are_those_of_the_children(P, sgs, lens, flags):
    """in fours from 2^20 on, where the arithmetic is the multiplied-out one unless a flag says otherwise: the scores that t + 1 steps leave, which
    are looked up, are the scores of the population that t steps leave, which reads them"""
    bits = sum(getattr(P, f) for f in flags.split("|") if f != "0")
    seg, tiles = lse_population(sgs, lens, seed=13)
    for steps in (1, 2):
        pop = dev(tiles)
        P.lse(sgs, seg, pop, 100, steps, 5, 52429, flags=bits)
        want = P.draft_score(sgs, seg, pop, flags=bits)
        got = P.lse(sgs, seg, dev(tiles), 100, steps + 1, 5, 52429, flags=bits)[0]
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (steps, int((got.view(torch.int32) != want.view(torch.int32)).sum()))
