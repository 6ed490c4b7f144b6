"""Selection where scores hold NaN (a model whose training diverged): they are ordered by their bits, above +infinity or, with the
sign bit, below -infinity, on every route, and every output row names one entry of its segment."""
import numpy as np
import pytest

from test_gpu_parity import P, dev  # noqa: F401  (P is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def by_bits(score, seg, k):
    u = score.view(np.uint32).astype(np.int64)
    u = np.where(u == 0x80000000, 0, u)
    key = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
    return np.stack([lo + np.argsort(-key[lo:hi], kind="stable")[:k] for lo, hi in zip(seg[:-1], seg[1:])]).astype(np.int32)


def scores(kind, n, rng):
    x = -np.exp2(rng.uniform(-26, -3, n)).astype(np.float32)
    u = x.view(np.uint32)
    some = rng.permutation(n)
    if kind == "one":
        u[some[:1]] = 0x7FC00000
    elif kind == "few of either sign":
        u[some[:9]], u[some[9:30]] = 0x7FC00001, 0xFFC00000
    elif kind == "many positive":
        u[some[: n // 3]] = 0x7FC00000
    elif kind == "many negative":
        u[some[: n - 20]] = 0xFFC00000
    elif kind == "payloads":
        u[some[: n // 2]] = 0x7F800001 + rng.integers(0, 0x7FFFFF, n // 2)
        u[some[n // 2: n - 9]] = 0xFF800001 + rng.integers(0, 0x7FFFFF, n - 9 - n // 2)
    elif kind == "all one":
        u[:] = 0xFFC00000
    elif kind == "last key":
        u[some[: n // 2]] = 0xFFFFFFFF
        u[some[n // 2:]] = 0x7FFFFFFF
    elif kind == "a crowded bin":   # the rest of it within one bin, in which lists hold their span's best
        x[:] = np.float32(1.0) + rng.integers(0, 1 << 16, n) * np.float32(2.0 ** -23)
        u[some[:40]], u[some[40: n // 50]] = 0x7FC00000, 0xFFC00000
    return x


@pytest.mark.parametrize("kind", ["one", "few of either sign", "many positive", "many negative", "payloads", "all one", "last key", "a crowded bin"])
@pytest.mark.parametrize("lens,ks", [([8000, 70], [1, 64]), ([4000, 300], [65, 300]), ([50001] * 3, [30, 512]), ([65536], [4096]), ([100001, 65537], [33, 4096]), ([500000], [512, 4096]),
                                     ([700001, 5000], [33, 4096]), ([3000001], [512]), ([1500] * 300, [100])])
def test_nan_by_its_bits(P, kind, lens, ks):
    rng = np.random.default_rng(len(kind) + sum(lens))
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    score = np.concatenate([scores(kind, n, rng) for n in lens])
    for k in ks:
        idx, val = P.topk(dev(score), seg, k)
        want = by_bits(score, seg, k)
        assert np.array_equal(idx.cpu().numpy(), want), (kind, k)
        assert np.array_equal(val.cpu().numpy().view(np.uint32), score.view(np.uint32)[want])


@pytest.mark.parametrize("n,k", [(300, 40), (4000, 65), (8000, 64), (30000, 300), (40000, 100), (65536, 3000), (100001, 1000), (270000, 100), (1100001, 1025), (3000001, 4096)])
def test_the_largest_word_of_all(P, n, k):
    """the largest key at index 0: a word of ones throughout is a word like any other"""
    score = (-np.exp2(np.random.default_rng(n).uniform(-26, -3, n))).astype(np.float32)
    bits = score.view(np.uint32)
    bits[0] = 0x7FFFFFFF
    seg = np.array([0, n], np.int64)
    want = by_bits(score, seg, k)
    idx, val = torch.full((1, k), -1, dtype=torch.int32, device="cuda"), torch.zeros((1, k), dtype=torch.float32, device="cuda")
    for call in (P.topk, P.topk_static):
        call(dev(score), seg, k, idx.fill_(-1), val.fill_(0))
        assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(val.cpu().numpy().view(np.uint32), bits[want])
