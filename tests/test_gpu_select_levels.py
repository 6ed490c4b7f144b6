"""Selections by the largest keys of blocks of 16, 64 and 256 neighbours: segment lengths around those at which a level is added, short
segments beside long ones, k from 1 to all blocks that are held, stretches of good entries, ties within and across blocks, NaN.
Against the oracle's stable sort, and with the maxima left by the draft kernel against the two separate calls."""
import ctypes as C

import numpy as np
import pytest

import workloads as w
from test_gpu_parity import P, dev  # noqa: F401  (P is a fixture)
from test_gpu_select_nan import by_bits, scores as with_nan
from test_gpu_select_shapes import check, of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CONV, GEMM, BATCHED = w.conv2d(1, 64, 56, 56, 64, 3, 3), w.gemm(512, 512, 512), w.batched_gemm(12, 128, 128, 64)


@pytest.mark.parametrize("kind", ["latencies", "ascending", "clump", "one bin", "two values", "300 values", "equal", "neighbours", "zeros"])
@pytest.mark.parametrize("lens,ks", [([32769], [1, 64, 768, 769, 1024]), ([40001, 16384, 16385, 1024], [65, 1024]), ([262144, 70], [3, 70]), ([262145, 16400], [512, 768, 769]),
                                     ([262161] * 3, [33]), ([1048576], [700]), ([1048577, 16385], [1, 768, 1000]), ([33000] * 129, [100, 256, 512]), ([700] * 60 + [300001, 4097] + [1000] * 60, [64, 500]), ([700, 4096, 8193] * 70 + [1100001] + [900] * 20, [300])])
def test_edges_of_the_levels(P, kind, lens, ks):
    rng = np.random.default_rng(len(kind) + len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)


@pytest.mark.parametrize("kind", ["latencies", "ascending", "nearly ascending", "clump", "clumps", "one bin", "two values", "300 values", "equal", "neighbours", "zeros"])
@pytest.mark.parametrize("lens,k", [([787200], 1025), ([787199], 1025), ([590592], 769), ([1200001, 1075200, 1075203, 1200002], 1400), ([1100001] * 5, 1400), ([3145728, 3145729], 4096), ([5000001], 2000), ([4194304], 64), ([4194305], 1), ([4194305, 600000], 768), ([4200003] * 2, 100)])
def test_few_of_long_segments(P, kind, lens, k):
    """lists of the parts of the best blocks of 256: one entry in 768 and one less, the most segments and one more"""
    rng = np.random.default_rng(len(kind) + len(lens))
    check(P, np.concatenate([of(kind, n, rng) for n in lens]), np.concatenate([[0], np.cumsum(lens)]), k)


@pytest.mark.parametrize("kind,n", [("latencies", 16777216), ("latencies", 16777217), ("ascending", 16777216)])
def test_the_longest_segments_by_blocks(P, kind, n):
    check(P, of(kind, n, np.random.default_rng(3)), np.array([0, n]), 4096)


def test_a_workspace_without_room_for_the_lists(P):
    """the query counts them for any k; with less another route serves"""
    score = torch.rand(2000000, device="cuda")
    seg = np.array([0, 900000, 2000000], np.int64)
    want, want_val = P.topk(score, seg, 1100)
    need = P.workspace_bytes(P.WS_TOPK, 2000000, 2, 1100)
    assert need == P.workspace_bytes(P.WS_TOPK, 2000000, 2, 1)
    ws = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
    idx, val = torch.empty_like(want), torch.empty_like(want_val)
    rc = P.load_library().pruner_topk(C.c_void_p(score.data_ptr()), seg.ctypes.data_as(C.POINTER(C.c_int64)), 2, 1100, C.c_void_p(idx.data_ptr()), C.c_void_p(val.data_ptr()),
                                      C.c_void_p(ws.data_ptr()), C.c_size_t(need - 256), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0 and torch.equal(idx, want) and torch.equal(val, want_val)


@pytest.mark.parametrize("k", [512, 1030])
def test_the_loop_in_a_workspace_for_other_calls(P, k):
    """one allocated for five subgraphs serves four and two, and one without room for the lists another route"""
    lens = [850001, 800003]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, sgs = int(seg[-1]), [GEMM, CONV]
    arr, start = P.to_c_subgraphs(sgs), P.random_init(sgs, seg, max(w.n_slots(s) for s in sgs), 9)
    need = P.workspace_bytes(P.WS_LSE, n, 2, k)
    for_five = P.workspace_bytes(P.WS_LSE, n, 5, k)
    assert need <= P.workspace_bytes(P.WS_LSE, n, 4, k) <= for_five
    want = None
    for size in (need, for_five, need - 256):
        tiles, score = start.clone(), torch.empty(n, dtype=torch.float32, device="cuda")
        spec_tiles, spec_score = torch.empty((tiles.shape[0], 2 * k), dtype=torch.uint16, device="cuda"), torch.empty(2 * k, dtype=torch.float32, device="cuda")
        count, ws = torch.empty(2, dtype=torch.int32, device="cuda"), torch.empty(size, dtype=torch.uint8, device="cuda")
        p = lambda t: C.c_void_p(t.data_ptr())
        rc = P.load_library().pruner_lse(arr, 2, seg.ctypes.data_as(C.POINTER(C.c_int64)), p(tiles), n, tiles.shape[0], 0, k, 3, 5, 40000, p(score), p(spec_tiles), p(spec_score), p(count),
                                         p(ws), C.c_size_t(size), C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        got = [t.cpu().numpy() for t in (tiles, score, spec_tiles, spec_score, count)]
        want = want or got
        assert all(np.array_equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("kind", ["few of either sign", "many negative", "payloads", "all one", "last key"])
def test_nan_among_the_parts(P, kind):
    rng = np.random.default_rng(len(kind))
    seg = np.array([0, 1100001, 2250002], np.int64)
    score = np.concatenate([with_nan(kind, n, rng) for n in np.diff(seg)])
    idx, val = P.topk(dev(score), seg, 1030)
    want = by_bits(score, seg, 1030)
    assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(val.cpu().numpy().view(np.uint32), score.view(np.uint32)[want])


@pytest.mark.parametrize("kind", ["few of either sign", "many positive", "many negative", "payloads", "all one", "last key"])
@pytest.mark.parametrize("lens", [[32769, 1100], [262145], [1048577]])
def test_nan_among_the_blocks(P, kind, lens):
    rng = np.random.default_rng(len(kind) + sum(lens))
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    score = np.concatenate([with_nan(kind, n, rng) for n in lens])
    for k in (30, 768, 1024):
        idx, val = P.topk(dev(score), seg, k)
        want = by_bits(score, seg, k)
        assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(val.cpu().numpy().view(np.uint32), score.view(np.uint32)[want])


@pytest.mark.parametrize("n_sg,n,k", [(90, 33000, 400), (90, 40000, 512), (130, 33000, 256), (130, 40000, 400), (130, 33000, 512)])
def test_nan_among_sorted_words(P, n_sg, n, k):
    """many segments, whose collections are sorted and not ranked: the surplus that the sort leaves out is found with NaN below the
    bound among the words, the scores spread over enough octaves that rank k's bin holds few"""
    rng = np.random.default_rng(n_sg + k)
    seg = np.arange(n_sg + 1, dtype=np.int64) * n
    score = (-np.exp2(rng.uniform(-20, -3, n_sg * n))).astype(np.float32)
    bits = score.view(np.uint32)
    for s in range(n_sg):
        some = s * n + rng.permutation(n)
        bits[some[:40]] = 0xFFC00000
        if s % 3 == 0:
            bits[some[40:45]] = 0x7FC00000
        if s % 5 == 0:
            bits[some[45:90]] = 0xFFFFFFFF
    idx, val = P.topk(dev(score), seg, k)
    want = by_bits(score, seg, k)
    assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(val.cpu().numpy().view(np.uint32), bits[want])


@pytest.mark.parametrize("n", [262161, 1048581, 1049601, 4194299])
def test_a_bound_below_every_number(P, n):
    """fewer than k blocks with anything but the least key of all, so that every block reaches the bound"""
    score = np.full(n, 0xFFFFFFFF, np.uint32).view(np.float32)
    score[np.random.default_rng(n).permutation(n)[:20]] = -1.5
    seg = np.array([0, n], np.int64)
    for k in (30, 256, 700):
        idx, val = P.topk(dev(score), seg, k)
        want = by_bits(score, seg, k)
        assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(val.cpu().numpy().view(np.uint32), score.view(np.uint32)[want])


@pytest.mark.parametrize("sgs,lens,k", [([GEMM], [16384], 500), ([GEMM], [16385], 500), ([GEMM], [70003], 1024), ([GEMM, CONV], [20001, 30003], 33), ([GEMM, CONV, BATCHED], [16386, 50001, 3], 3),
                                        ([GEMM, CONV, BATCHED], [300001, 200003, 120002], 700), ([CONV, GEMM], [1048580, 17001], 1000), ([CONV], [1048576], 64), ([GEMM], [40000], 4096),
                                        ([CONV, GEMM, GEMM], [1700001, 900002, 50], 50), ([GEMM, CONV], [1200003, 1100001], 1050), ([CONV], [22399], 700), ([CONV], [22400], 700),
                                        ([CONV, GEMM], [65537, 20001], 768), ([GEMM, CONV] * 45, [17000] * 90, 399), ([GEMM, CONV] * 45, [17000] * 90, 400)])
def test_maxima_left_by_the_draft_kernel(P, sgs, lens, k):
    """one candidate per thread and four, ends of segments inside a block, a population with few distinct scores (GEMM)"""
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    tiles = P.random_init(sgs, seg, max(w.n_slots(s) for s in sgs), 23)
    for flags in (P.REFERENCE_ROUNDING, P.FUSED_ARITHMETIC):
        score, idx, val = P.prior_filter(sgs, seg, tiles, k, flags=flags)
        want, want_val = P.topk(score, seg, k)
        assert torch.equal(idx, want) and torch.equal(val.view(torch.int32), want_val.view(torch.int32))
        host = score.cpu().numpy()
        assert np.array_equal(idx.cpu().numpy(), by_bits(host, seg, k))


@pytest.mark.parametrize("longest", [512, 513, 2048, 2049, 4096, 4097, 8192])
@pytest.mark.parametrize("kind", ["latencies", "ascending", "two values", "equal"])
def test_words_per_thread_of_short_selections(P, longest, kind):
    rng = np.random.default_rng(longest)
    lens = [longest, 64, longest - 1]
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in (1, 33, 64):
        check(P, score, seg, k)
