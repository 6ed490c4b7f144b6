"""pruner_lse on short segments at the lines between its routes: one workgroup per subgraph with 8, 16 or 32 keys a thread, or the launches
over the whole device (long segments, or more than 512 members of S_spec, where subgraphs and members are few).  Against the
oracle's loop, every integer and every bit of the scores."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, check_lse_against_oracle, lse_population  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

GEMM = w.gemm(96, 80, 72, hw=w.toy_device())
CONV = w.conv2d(1, 8, 12, 12, 16, 3, 3)
BATCHED = w.batched_gemm(4, 32, 48, 40)


@pytest.mark.parametrize("k", [64, 512, 513])
@pytest.mark.parametrize("n", [8193, 16383, 16384, 16385])
def test_keys_per_thread(P, n, k):
    seg, tiles = lse_population([CONV], [n], seed=n + k)
    check_lse_against_oracle(P, [CONV], seg, tiles, k, 3, 7 + k, 52000)


@pytest.mark.parametrize("n_sg", [7, 8])
def test_more_members_than_half_the_threads(P, n_sg):
    """520 members: 7 subgraphs stay below the line, 8 do not; all entries of a segment are chosen in the first"""
    sgs = [GEMM, CONV, BATCHED, GEMM, BATCHED, CONV, GEMM, GEMM][:n_sg]
    lens = [520, 1303, 900, 2049, 521, 777, 1600, 640][:n_sg]
    seg, tiles = lse_population(sgs, lens, seed=n_sg)
    check_lse_against_oracle(P, sgs, seg, tiles, 520, 3, 11, 52429)


@pytest.mark.parametrize("n_sg", [20, 21])
def test_long_segments_of_many_subgraphs(P, n_sg):
    """k = 1,000: 20 subgraphs stay below the line, 21 do not"""
    sgs = [GEMM] * n_sg
    seg, tiles = lse_population(sgs, [16401] + [1500] * (n_sg - 1), seed=n_sg)
    check_lse_against_oracle(P, sgs, seg, tiles, 1000, 2, 13, 52429)


@pytest.mark.parametrize("n_sg", [78, 79])
def test_a_long_segment_among_many_short_ones(P, n_sg):
    """k = 8 beside one of 16,400: 78 subgraphs stay below the line, 79 do not"""
    sgs = [GEMM, BATCHED] * (n_sg // 2) + [GEMM] * (n_sg % 2)
    seg, tiles = lse_population(sgs, [16400] + [300 + i % 5 for i in range(n_sg - 1)], seed=n_sg)
    check_lse_against_oracle(P, sgs, seg, tiles, 8, 3, 17, 52429)


@pytest.mark.parametrize("n,k", [(720, 703), (720, 704), (1536, 600), (1537, 600)])
def test_members_above_half_the_threads_of_short_segments(P, n, k):
    seg, tiles = lse_population([CONV], [n], seed=n + k)
    check_lse_against_oracle(P, [CONV], seg, tiles, k, 3, 19, 52429)


def test_copies_in_either_kernel(P):
    """five schedules over and over: ties at rank k by the thousand, with 16 keys a thread and by the launches over the device"""
    for n in (16000, 17000):
        seg, tiles = lse_population([GEMM], [n], seed=3)
        tiles[:, 5:] = tiles[:, np.arange(n - 5) % 5]
        check_lse_against_oracle(P, [GEMM], seg, tiles, 300, 3, 12, 60000)
