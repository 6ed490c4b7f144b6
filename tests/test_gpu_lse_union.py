"""pruner_lse on segments too long for one launch per step, where the union of S_spec and the k best is formed by three launches
over the whole device: S_spec sizes around a wavefront's, a workgroup's and the largest, several subgraphs side by side, and
populations of copies (scores shared by whole lists; a union with fewer schedules than k).  Against the oracle's loop, every
integer and every bit of the scores."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, check_lse_against_oracle, lse_population  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

GEMM = w.gemm(96, 80, 72, hw=w.toy_device())
FRAG = w.gemm(64, 64, 64, dtype_bytes=2, hw=w.toy_device(), rd_levels=3, frag=(16, 16, 16))
CONV = w.conv2d(1, 8, 12, 12, 16, 3, 3)


@pytest.mark.parametrize("k", [1, 15, 17, 63, 64, 65, 1023, 1025, 4095, 4096])
def test_one_segment(P, k):
    seg, tiles = lse_population([CONV], [32772], seed=k)
    check_lse_against_oracle(P, [CONV], seg, tiles, k, 3, k, 50000)


@pytest.mark.parametrize("k", [30, 1200])
def test_several_segments(P, k):
    sgs = [GEMM, CONV, FRAG]
    seg, tiles = lse_population(sgs, [33001, 1201, 4098], seed=2)
    check_lse_against_oracle(P, sgs, seg, tiles, k, 4, 9, 52000)


@pytest.mark.parametrize("distinct,q16", [(1, 0), (3, 0), (700, 0), (700, 60000), (5000, 20000)])
def test_a_population_of_copies(P, distinct, q16):
    seg, tiles = lse_population([GEMM], [33000], seed=3)
    tiles[:, distinct:] = tiles[:, np.arange(33000 - distinct) % distinct]
    check_lse_against_oracle(P, [GEMM], seg, tiles, 2048, 3, 12, q16)


def test_many_segments(P):
    """as many subgraphs as make the union's workgroups take 256 places each"""
    lens = [1100 + 4 * (t % 7) for t in range(64)]
    sgs = [GEMM, CONV] * 32
    seg, tiles = lse_population(sgs, lens, seed=5)
    check_lse_against_oracle(P, sgs, seg, tiles, 1030, 3, 11, 40000)


@pytest.mark.parametrize("n_sg,k,distinct", [(17, 2050, 3000), (40, 4096, 100), (40, 4096, 4200), (260, 1025, 1300)])
def test_several_groups_per_ranking_workgroup(P, n_sg, k, distinct):
    """two, five and eight groups of 64 entries: groups of S_spec and of the k best in one workgroup, S_spec of few members, a last
    workgroup with fewer groups, and a k that no multiple of 64 is"""
    lens = [k + 4 * (t % 5) for t in range(n_sg)]
    sgs = [GEMM if t % 2 else FRAG for t in range(n_sg)]
    seg, tiles = lse_population(sgs, lens, seed=n_sg)
    for t in range(n_sg):
        mine = tiles[:, seg[t]:seg[t + 1]]
        mine[:, distinct:] = mine[:, np.arange(max(0, lens[t] - distinct)) % distinct]
    check_lse_against_oracle(P, sgs, seg, tiles, k, 3, 13, 30000)
