"""pruner_lse where the chosen children are made again, 64 to a workgroup: k on both sides of whole workgroups, extents with large primes
(a long search for a child's prime factors) beside powers of two.  Against the oracle's loop, every integer and every bit of the scores."""
import pytest

import workloads as w
from test_gpu_parity import P, check_lse_against_oracle, lse_population  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu

PRIMES = w.gemm(46337, 1031, 61, hw=w.toy_device())
POWERS = w.gemm(512, 512, 512)


@pytest.mark.parametrize("k", [1025, 1087, 1088, 1089])
@pytest.mark.parametrize("sgs", [[PRIMES], [PRIMES, POWERS]], ids=["primes", "both"])
def test_chosen_children(P, sgs, k):
    seg, tiles = lse_population(sgs, [1100, 1090][: len(sgs)], seed=k)
    check_lse_against_oracle(P, sgs, seg, tiles, k, 3, 5, 60000)


@pytest.mark.parametrize("k", [1, 63, 64, 65])
def test_few_of_a_long_segment(P, k):
    seg, tiles = lse_population([POWERS], [33001], seed=k)
    check_lse_against_oracle(P, [POWERS], seg, tiles, k, 3, 6, 50000)
