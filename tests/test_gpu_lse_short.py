"""pruner_lse on short segments, where one launch per step selects from S_x and forms the new S_spec: segment lengths around a
thread's share of the entries, S_spec sizes around a wavefront's and at both ends of the route's range, populations of copies
(ties to be taken in index order), one and two loop-nest classes (children made in the draft kernels) and more or unaligned
ones (the mutation as a launch of its own).  Against the oracle's loop, every integer and every bit of the scores."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, check_lse_against_oracle, lse_population  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

GEMM = w.gemm(96, 80, 72, hw=w.toy_device())
FRAG = w.gemm(64, 64, 64, dtype_bytes=2, hw=w.toy_device(), rd_levels=3, frag=(16, 16, 16))
CONV = w.conv2d(1, 8, 12, 12, 16, 3, 3)
BATCHED = w.batched_gemm(4, 32, 48, 40)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 512, 1000, 1024])
@pytest.mark.parametrize("lens", [[1024], [1028], [8192], [8196], [32768]])
def test_one_segment(P, lens, k):
    seg, tiles = lse_population([GEMM], lens, seed=31 + k)
    check_lse_against_oracle(P, [GEMM], seg, tiles, min(k, lens[0]), 3, 5 + k, 50000)


@pytest.mark.parametrize("sgs,lens", [([GEMM, BATCHED], [4000, 2056]), ([GEMM, CONV, BATCHED], [4000, 1200, 2056]),
                                      ([CONV, GEMM, FRAG], [1001, 999, 1502]), ([FRAG, FRAG, GEMM], [9000, 64, 64])])
def test_several_segments(P, sgs, lens):
    seg, tiles = lse_population(sgs, lens, seed=8)
    check_lse_against_oracle(P, sgs, seg, tiles, 60, 4, 99, 52000)


@pytest.mark.parametrize("n", [8192, 20000])
def test_a_population_of_copies(P, n):
    """five schedules over and over: the rank-k key is shared by thousands, and the union keeps five schedules at first"""
    seg, tiles = lse_population([GEMM], [n], seed=3)
    tiles[:, 5:] = tiles[:, np.arange(n - 5) % 5]
    check_lse_against_oracle(P, [GEMM], seg, tiles, 700, 3, 12, 60000)
    check_lse_against_oracle(P, [GEMM], seg, tiles, 700, 2, 12, 0)


def test_the_longest_segment_of_the_route_and_one_entry_more(P):
    for n in (32768, 32772):
        seg, tiles = lse_population([CONV], [n], seed=6)
        check_lse_against_oracle(P, [CONV], seg, tiles, 1024, 2, 4, 40000)
    seg, tiles = lse_population([CONV], [6000], seed=6)
    check_lse_against_oracle(P, [CONV], seg, tiles, 1025, 2, 4, 40000)
