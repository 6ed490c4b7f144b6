"""The selection's first digit (narrow bins inside a window of octaves, wide ones outside, either sign) and its routes behind
that digit: lengths around the edges of a sweep and of the one-launch route, k at both ends, values in and around the window,
collections that fit, that fit after the bin is split, and ties that do not fit at all.  Against the oracle's stable sort."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import P, dev  # noqa: F401  (P is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(P, score, seg, k):
    seg = np.asarray(seg, np.int64)
    idx, val = P.topk(dev(score), seg, k)
    torch.cuda.synchronize()
    want, want_val = oracle.topk(score, seg, k)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(val.cpu().numpy().view(np.uint32), np.asarray(want_val, np.float32).view(np.uint32))
    if len(seg) <= 17:
        i2, v2 = torch.empty_like(idx), torch.empty_like(val)
        P.topk_static(dev(score), seg, k, i2, v2)
        assert torch.equal(i2, idx) and torch.equal(v2.view(torch.int32), val.view(torch.int32))


def values(kind, n, rng):
    x = rng.standard_normal(n)
    if kind == "normal":
        return x.astype(np.float32)
    if kind == "latencies":
        return (-np.exp2(rng.uniform(-26, -3, n))).astype(np.float32)
    if kind == "every exponent":       # both signs, denormals to the largest
        return (np.sign(x) * np.exp2(rng.uniform(-149, 127.9, n))).astype(np.float32)
    if kind == "tiny":                 # below any window
        return (np.sign(x) * np.exp2(rng.uniform(-140, -30, n))).astype(np.float32)
    if kind == "huge":                 # above any window, infinities among them
        y = (np.sign(x) * np.exp2(rng.uniform(20, 127, n))).astype(np.float32)
        y[rng.integers(0, n, n // 50 + 1)] = np.inf
        y[rng.integers(0, n, n // 50 + 1)] = -np.inf
        return y
    if kind == "zeros":                # zeros of either sign, few others
        y = np.where(rng.random(n) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
        y[rng.integers(0, n, n // 100 + 1)] = 1e-38
        y[rng.integers(0, n, n // 100 + 1)] = -1e-45
        return y
    if kind == "one bin":              # all within a three-per-cent bin: the digits behind the first decide
        return np.float32(1.0) + (rng.integers(0, 1 << 16, n) * np.float32(2.0 ** -23)).astype(np.float32)
    if kind == "two values":
        return np.where(rng.random(n) < 0.3, np.float32(-0.25), np.float32(-0.75)).astype(np.float32)
    if kind == "window edges":         # the powers of two where bins change width, and their neighbours
        e = np.exp2(np.array([-24, -23, -22, -10, -11, -7, -6, -5, 6, 7, 8, 10, 11, 12], np.float64))
        y = (rng.choice(e, n) * rng.choice([1, -1], n)).astype(np.float32)
        return np.nextafter(y, np.float32(rng.choice([-1, 1]) * 1e30)).astype(np.float32) if rng.random() < 0.5 else y
    if kind == "300 values":           # every value shared by a few hundred to a few thousand
        return (-1.0 - rng.integers(0, 300, n) / 8).astype(np.float32)
    if kind == "one value a bin":      # ties that fill a bin, others in the bins beside it
        return np.where(rng.random(n) < 0.05, np.float32(2.0), (0.5 * x).astype(np.float32)).astype(np.float32)
    return np.full(n, np.float32(-3.5))


KINDS = ["normal", "latencies", "every exponent", "tiny", "huge", "zeros", "one bin", "two values", "window edges", "300 values", "one value a bin", "equal"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("lens,ks", [([8193], [1, 64, 65, 4096]), ([16383, 16384, 16385, 70], [1, 33, 70]), ([65536], [1, 512, 4096]), ([65535, 5, 32769], [5]),
                                     ([65537], [1, 31, 4096]), ([300001], [100, 4096]), ([50001] * 7, [512]), ([333333] * 3, [33, 512]), ([524288, 524287], [4096]), ([524289], [1, 4096]),
                                     ([540001, 600000, 33], [33]), ([3000001], [512, 4096])])
def test_routes_and_values(P, kind, lens, ks):
    rng = np.random.default_rng(sum(lens) + len(kind))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([values(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)


def test_more_segments_than_compute_units(P):
    rng = np.random.default_rng(0)
    lens = rng.integers(90, 9000, size=300)
    seg = np.concatenate([[0], np.cumsum(lens)])
    check(P, values("latencies", int(seg[-1]), rng), seg, 90)
