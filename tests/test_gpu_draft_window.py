"""Draft scores of populations that are column windows of a wider matrix: the same bits as from a copy of the window, whatever the
window's first column and length, also where it ends at the matrix's right edge."""
import ctypes as C

import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, dev  # noqa: F401  (P is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SUBGRAPHS = [w.gemm(512, 512, 512), w.conv2d(1, 64, 56, 56, 64, 3, 3), w.batched_gemm(12, 128, 128, 64)]


def _window_scores(P, sgs, seg, matrix, column, flags):
    lib, n = P.load_library(), int(seg[-1])
    seg = np.asarray(seg, np.int64)
    score = torch.full((n + 8,), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.empty(P.workspace_bytes(P.WS_DRAFT, n, len(sgs), 0), dtype=torch.uint8, device="cuda")
    rc = lib.pruner_draft_score(P.to_c_subgraphs(sgs), len(sgs), seg.ctypes.data_as(C.POINTER(C.c_int64)), matrix.data_ptr() + 2 * column, matrix.shape[1],
                                flags, score.data_ptr(), None, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = score.cpu().numpy()
    assert np.all(got[n:] == 7.0)
    return got[:n].view(np.uint32)


@pytest.mark.parametrize("column,lens", [(5, [1000]), (5, [1001]), (3, [1002]), (1, [1003]), (0, [9]), (5, [2]), (7, [3]), (6, [4]), (2, [5]), (5, [700, 301]),
                                         (9, [401, 3, 597])])
def test_a_window_scores_like_its_copy(P, column, lens):
    sgs = SUBGRAPHS[: len(lens)]
    seg = np.concatenate([[0], np.cumsum(lens)])
    n, rows = int(seg[-1]), max(w.n_slots(s) for s in sgs)
    tiles = np.ones((rows, column + n), np.uint16)
    for t, sg in enumerate(sgs):
        tl, _ = w.sample_population(sg, lens[t], seed=9, stream=t)
        tiles[: tl.shape[0], column + seg[t]:column + seg[t + 1]] = tl
    matrix = dev(tiles)
    for flags in (P.REFERENCE_ROUNDING, P.FUSED_ARITHMETIC):
        copy = P.draft_score(sgs, seg, dev(tiles[:, column:]), flags=flags).cpu().numpy().view(np.uint32)
        assert np.array_equal(_window_scores(P, sgs, seg, matrix, column, flags), copy)


@pytest.mark.parametrize("n", [1, 2, 3])
def test_the_single_loads_of_tiny_populations_give_the_wide_loads_bits(P, n):
    """Fewer than four candidates are loaded one by one, whatever the pitch: the same bits as from the same candidates among a
    thousand, symbols included, and the selection behind them is that of the two calls."""
    shapes = SUBGRAPHS + [w.depthwise_conv2d(1, 512, 28, 28, 3, 3), w.gemm(1024, 256, 256, dtype_bytes=2, rd_levels=3, frag=(16, 16, 16))]
    for sg in shapes:
        wide, _ = w.sample_population(sg, 1000, seed=4)
        for flags in (P.REFERENCE_ROUNDING, P.FUSED_ARITHMETIC):
            score, sym = P.draft_score([sg], [0, 1000], dev(wide), flags=flags, symbols=True)
            for pitch in (n, n + 1, 9):
                narrow = dev(wide[:, :pitch])
                few, few_sym = P.draft_score([sg], [0, n], narrow, flags=flags, symbols=True)
                assert torch.equal(few.view(torch.int32), score[:n].view(torch.int32)) and torch.equal(few_sym, sym[:, :n])
                plain = P.draft_score([sg], [0, n], narrow, flags=flags)
                assert torch.equal(plain.view(torch.int32), few.view(torch.int32))
                filtered, idx, val = P.prior_filter([sg], [0, n], narrow, n, flags=flags)
                want, want_val = P.topk(few, [0, n], n)
                assert torch.equal(filtered.view(torch.int32), few.view(torch.int32)) and torch.equal(idx, want) and torch.equal(val, want_val)
