"""pruner_pacm_score where its tiles of whole candidates can go wrong: candidates of one row (a tile is then full by count, not
by rows), of eight, of none, runs of either next to each other, sets at the edges of a group and of a wavefront's share; candidates
wherever they may lie, candidates with infinite or NaN features, which must not reach their neighbours, and infinite biases."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w
from test_gpu_parity import P, check_pacm, dev, gpu_pacm, pacm_tolerance  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


def _counts(kind, n_d, rng):
    if kind == "ones":
        return np.ones(n_d, np.int32)
    if kind == "eights":
        return np.full(n_d, 8, np.int32)
    if kind == "runs":   # none, many, one, in runs longer than a tile
        return np.repeat(np.array([0, 8, 1, 5, 0, 3], np.int32), 40)[np.arange(n_d) % 240]
    return rng.integers(0, 9, size=n_d).astype(np.int32)


@pytest.mark.parametrize("n_d", [1, 31, 33, 257, 8 * 256 + 1, 20000])
@pytest.mark.parametrize("stmt,blk", [("ones", "eights"), ("eights", "ones"), ("runs", "runs"), ("mixed", "mixed")])
def test_tiles_of_whole_candidates(P, n_d, stmt, blk):
    rng = np.random.default_rng(n_d)
    m = w.make_pacm_weights(seed=4)
    n_stmt, n_blk = _counts(stmt, n_d, rng), _counts(blk, n_d, rng)[::-1].copy()
    ids = np.arange(n_d) * 7 + 2
    feat = w.make_statement_features(ids, n_stmt, pad_value=np.float32("nan"))
    flow = w.make_flow_features(ids, n_blk, pad_value=np.float32("inf"))
    if n_d <= 3000:
        check_pacm(P, feat, n_stmt, flow, n_blk, m, label=f"{n_d} {stmt} {blk}")
        return
    got = P.pacm_score(dev(feat), dev(n_stmt), dev(flow), dev(n_blk), gpu_pacm(m)).cpu().numpy()
    pick = rng.choice(n_d, size=1500, replace=False)
    want, _ = oracle.pacm(feat[pick], n_stmt[pick], flow[pick], n_blk[pick], m)
    assert np.all(np.abs(got[pick] - want) <= pacm_tolerance(want))


def _score(P, feat, n_stmt, flow, n_blk, gm):
    return P.pacm_score(dev(feat), dev(n_stmt), dev(flow), dev(n_blk), gm).cpu().numpy().view(np.uint32)


def test_a_score_is_a_function_of_its_candidate_alone(P):
    """The same bits from a set that is cut elsewhere, where a candidate's rows begin at another place of a tile and go to other
    workgroups, and from candidates of every count scored one by one."""
    rng = np.random.default_rng(8)
    gm = gpu_pacm(w.make_pacm_weights(seed=6))
    n_d = 20000
    n_stmt, n_blk = rng.integers(0, 9, size=n_d).astype(np.int32), rng.integers(0, 9, size=n_d).astype(np.int32)
    ids = rng.permutation(n_d)
    feat, flow = w.make_statement_features(ids, n_stmt), w.make_flow_features(ids, n_blk)
    whole = _score(P, feat, n_stmt, flow, n_blk, gm)
    for lo, hi in ((1, n_d), (2, 9000), (3, 3004), (8, n_d - 1), (9, 520), (4001, n_d)):
        assert np.array_equal(_score(P, feat[lo:hi], n_stmt[lo:hi], flow[lo:hi], n_blk[lo:hi], gm), whole[lo:hi]), (lo, hi)
    for count in range(81):
        i = int(np.flatnonzero((n_stmt == count // 9) & (n_blk == count % 9))[-1])
        assert np.array_equal(_score(P, feat[i:i + 1], n_stmt[i:i + 1], flow[i:i + 1], n_blk[i:i + 1], gm), whole[i:i + 1]), count


@pytest.mark.parametrize("what", [np.inf, np.nan, 3e38])
def test_a_candidate_with_special_features_stays_by_itself(P, what):
    """A candidate's score is the same bits whether or not its neighbours' features are finite, and those of a candidate with
    special features are the ones it gets alone."""
    rng = np.random.default_rng(3)
    n_d = 700
    gm = gpu_pacm(w.make_pacm_weights(seed=5))
    n_stmt, n_blk = rng.integers(1, 9, size=n_d).astype(np.int32), rng.integers(1, 9, size=n_d).astype(np.int32)
    ids = np.arange(n_d) + 11
    feat, flow = w.make_statement_features(ids, n_stmt), w.make_flow_features(ids, n_blk)
    clean = _score(P, feat, n_stmt, flow, n_blk, gm)
    assert np.isfinite(clean.view(np.float32)).all()
    bad_s, bad_b = np.arange(5, n_d, 37), np.arange(9, n_d, 41)
    feat[bad_s, 0, ::5] = what
    flow[bad_b, 0, ::3] = what
    got = _score(P, feat, n_stmt, flow, n_blk, gm)
    special = np.union1d(bad_s, bad_b)
    others = np.setdiff1d(np.arange(n_d), special)
    assert np.array_equal(got[others], clean[others])
    for i in special:
        assert np.array_equal(got[i:i + 1], _score(P, feat[i:i + 1], n_stmt[i:i + 1], flow[i:i + 1], n_blk[i:i + 1], gm))


@pytest.mark.parametrize("value", [-np.inf, -3.4e38])
def test_a_bias_of_minus_infinity_switches_its_unit_off(P, value):
    """The bias is a binary32 addend: relu makes 0 of minus infinity, and of a finite value that is infinite in bfloat16."""
    rng = np.random.default_rng(2)
    n_d = 300
    m = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in w.make_pacm_weights(seed=7).items()}
    m["b1"][::9] = value
    m["be"][::7] = value
    n_stmt, n_blk = rng.integers(0, 9, size=n_d).astype(np.int32), rng.integers(0, 9, size=n_d).astype(np.int32)
    ids = np.arange(n_d) + 3
    check_pacm(P, w.make_statement_features(ids, n_stmt), n_stmt, w.make_flow_features(ids, n_blk), n_blk, m, label=f"bias {value}")
