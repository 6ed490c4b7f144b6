"""Selections at the edges of the one- and two-launch routes' ways of ranking and collecting: one launch for everything (segments of
up to 32,768), words ranked in rounds or sorted, with or without the last bin's surplus, stretches of good entries that
overflow a span's list.  Against the oracle's stable sort."""
import numpy as np
import pytest

from test_gpu_parity import P  # noqa: F401  (a fixture)
from test_gpu_select_digits import check, values

pytestmark = pytest.mark.gpu


def of(kind, n, rng):
    if kind in ("ascending", "descending"):
        x = np.sort(values("latencies", n, rng))
        return x if kind == "ascending" else x[::-1].copy()
    if kind == "clump":   # a stretch of good entries in the middle, in no order
        x = values("latencies", n, rng)
        m = min(n, 3000)
        x[n // 2 - m // 2: n // 2 - m // 2 + m] = -np.exp2(rng.uniform(-30, -27, m)).astype(np.float32)
        return x
    if kind == "nearly ascending":      # one in fifty elsewhere
        x = np.sort(values("latencies", n, rng))
        some = rng.integers(0, n, n // 50 + 1)
        x[some] = x[some[::-1]]
        return x
    if kind == "clumps":                # good entries side by side in five places
        x = values("latencies", n, rng)
        for p in range(5):
            x[p * (n // 7): p * (n // 7) + 3000] *= np.float32(2.0 ** -10)
        return x
    if kind == "ties and neighbours":   # a third of the entries share a value, a few lie just above it
        r = rng.random(n)
        return np.where(r < 0.3, np.float32(2.0), np.where(r < 0.3005, np.float32(2.0) + (r * 0.01).astype(np.float32), values("normal", n, rng) * np.float32(0.3))).astype(np.float32)
    if kind == "neighbours":            # one bin: mostly one value, a few just above it
        return (np.float32(2.0) + (rng.random(n) < 0.0001) * rng.integers(1, 5, n) * np.float32(2.0 ** -22)).astype(np.float32)
    return values(kind, n, rng)


@pytest.mark.parametrize("kind", ["ascending", "clump", "one bin", "300 values", "equal", "ties and neighbours", "two values"])
@pytest.mark.parametrize("lens,ks", [([100001, 65537], [3, 512, 1100, 1280, 1281, 4096]), ([300001] * 3, [33, 2048]), ([524288], [512, 4096]), ([70000] * 130, [512])])
def test_lists_that_overflow(P, kind, lens, ks):
    rng = np.random.default_rng(len(kind) + len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)


@pytest.mark.parametrize("kind", ["one bin", "neighbours", "two values", "300 values", "ascending"])
@pytest.mark.parametrize("lens,ks", [([524288], [1, 40, 128, 129, 1279, 1280, 1281]), ([480001] * 18, [40]), ([300001, 200000, 524287, 196608, 196609, 294912, 294914], [2, 128, 900])])
def test_lists_of_a_crowded_bin(P, kind, lens, ks):
    """around 12 and 18 spans' worth of entries in the bin, spans of one sweep and of two, the k best of a span with and without
    ties that fill it"""
    rng = np.random.default_rng(len(kind) + len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)


@pytest.mark.parametrize("kind", ["latencies", "ascending", "descending", "one bin", "two values", "300 values", "equal"])
@pytest.mark.parametrize("lens,ks", [([40000] * 20, [4096]), ([33000] * 130, [65, 512, 2047, 2048]), ([65536] * 40, [1023, 4096]), ([32769, 5000], [4096]), ([40000] * 300, [600])])
def test_sorted_or_ranked(P, kind, lens, ks):
    rng = np.random.default_rng(len(kind) + len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)


@pytest.mark.parametrize("kind", ["latencies", "ascending", "every exponent", "zeros", "one bin", "two values", "300 values", "equal"])
@pytest.mark.parametrize("lens,ks", [([65], [65]), ([66, 67, 4095], [65, 66]), ([4096], [65, 4096]), ([4097, 4100], [512, 4096]), ([8192], [1000]), ([32768], [1, 70, 4096]), ([32767, 70, 2], [1, 2]),
                                     ([32768, 16385, 70], [70]), ([500] * 129, [100]), ([2000] * 300, [512]), ([5000] * 140, [4096])])
def test_one_launch(P, kind, lens, ks):
    rng = np.random.default_rng(len(kind) + len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)])
    score = np.concatenate([of(kind, n, rng) for n in lens])
    for k in ks:
        check(P, score, seg, k)
