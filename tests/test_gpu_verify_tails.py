"""pruner_verify_score where a workgroup's last tile has up to 32 rows, which is taken without a second half: totals on both sides of 32
and 64 rows, alone and behind a whole tile, and a candidate whose rows run on from the whole tile into the last one."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, check_verify  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


def counts_of(total, n):
    """n counts of 0..8 that add up to total"""
    out = np.zeros(n, np.int32)
    for i in range(n):
        out[i] = min(8, total - out.sum())
    return out


@pytest.mark.parametrize("rows", [1, 7, 31, 32, 33, 63, 64])
def test_one_tile(P, rows):
    n_stmt = counts_of(rows, 8)
    check_verify(P, w.make_statement_features(np.arange(8) * 3 + 1, n_stmt, pad_value=1e6), n_stmt, w.make_mlp_weights(seed=2))


@pytest.mark.parametrize("first", [57, 61, 64])
@pytest.mark.parametrize("second", [1, 8, 31, 32, 35, 36, 39, 40, 64])
def test_behind_a_whole_tile(P, first, second):
    """2,056 candidates: the first workgroup alone has sixteen, its rows those of two groups of eight"""
    n_d = 2056
    n_stmt = np.random.default_rng(first + second).integers(0, 3, size=n_d).astype(np.int32)
    n_stmt[:8], n_stmt[2048:] = counts_of(first, 8), counts_of(second, 8)
    check_verify(P, w.make_statement_features(np.arange(n_d) * 7 + 2, n_stmt, pad_value=-2e5), n_stmt, w.make_mlp_weights(seed=3))
