"""Small populations are drawn in one launch whose argument holds the tables, larger ones and those with more tables by tables of
factors: the oracle's bits from either, at the edges of the rule."""
import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, oracle  # noqa: F401  (P is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CONV, GEMM = w.conv2d(1, 64, 56, 56, 64, 3, 3), w.gemm(512, 512, 512)
FRAGMENTS = w.gemm(1024, 256, 256, dtype_bytes=2, rd_levels=3, frag=(16, 16, 16))


@pytest.mark.parametrize("sgs,lens", [([GEMM], [1]), ([GEMM], [255]), ([CONV], [65536]), ([CONV], [65537]), ([GEMM, CONV, FRAGMENTS], [30001, 0, 35535]), ([GEMM, CONV, FRAGMENTS], [257, 1, 513]),
                                      ([CONV, GEMM, FRAGMENTS] * 4, [101] * 12), ([w.gemm(64 * (i % 30 + 1), 96, 128) for i in range(60)], [33] * 60)])
def test_one_launch_and_three(P, sgs, lens):
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, rows = int(seg[-1]), max(w.n_slots(s) for s in sgs) + 1
    tiles = torch.full((rows, n + 3), 0xFFFF, dtype=torch.uint16, device="cuda")
    P.random_init(sgs, seg, rows, 41, tiles=tiles)
    got = tiles.cpu().numpy()
    assert np.array_equal(got[:, :n], oracle.random_init(sgs, seg, rows, seed=41)) and (got[:, n:] == 0xFFFF).all()


@pytest.mark.parametrize("lens,pad", [([1048576], 0), ([524289, 0, 524290], 5), ([7, 1048000, 590], 3), ([1048577], 3)])
def test_eight_candidates_per_thread(P, lens, pad):
    """from 2^20 candidates on, rows of whole groups of eight; ragged segments, and a pitch that leaves groups of four (the last)"""
    sgs = [CONV, FRAGMENTS, GEMM][: len(lens)]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, rows = int(seg[-1]), max(w.n_slots(s) for s in sgs) + 1
    tiles = torch.full((rows, (n + pad) // 4 * 4), 0xFFFF, dtype=torch.uint16, device="cuda")
    P.random_init(sgs, seg, rows, 43, tiles=tiles)
    got = tiles.cpu().numpy()
    assert np.array_equal(got[:, :n], oracle.random_init(sgs, seg, rows, seed=43)) and (got[:, n:] == 0xFFFF).all()
