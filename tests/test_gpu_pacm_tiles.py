"""pruner_pacm_score where its tiles of whole candidates can go wrong: candidates of one row (a tile is then full by count, not
by rows), of eight, of none, runs of either next to each other, sets at the edges of a group and of a wavefront's share; and
candidates with infinite or NaN features, which must not reach their neighbours."""
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


@pytest.mark.parametrize("what", [np.inf, np.nan, 3e38])
def test_a_candidate_with_special_features_stays_by_itself(P, what):
    """A candidate's score is the same whether or not its neighbours' features are finite.  The sums over its rows are taken
    in the same order either way (the other candidates' rows contribute zeros), so the bits agree."""
    rng = np.random.default_rng(3)
    n_d = 700
    m = w.make_pacm_weights(seed=5)
    n_stmt, n_blk = rng.integers(1, 9, size=n_d).astype(np.int32), rng.integers(1, 9, size=n_d).astype(np.int32)
    ids = np.arange(n_d) + 11
    feat, flow = w.make_statement_features(ids, n_stmt), w.make_flow_features(ids, n_blk)
    clean = P.pacm_score(dev(feat), dev(n_stmt), dev(flow), dev(n_blk), gpu_pacm(m)).cpu().numpy()
    bad_s, bad_b = np.arange(5, n_d, 37), np.arange(9, n_d, 41)
    feat[bad_s, 0, ::5] = what
    flow[bad_b, 0, ::3] = what
    got = P.pacm_score(dev(feat), dev(n_stmt), dev(flow), dev(n_blk), gpu_pacm(m)).cpu().numpy()
    others = np.setdiff1d(np.arange(n_d), np.concatenate([bad_s, bad_b]))
    assert np.isfinite(clean).all()
    assert np.abs(got[others] - clean[others]).max() <= pacm_tolerance(clean).min()
    assert (np.abs(got[others] - clean[others]) <= 1e-5 * np.abs(clean).max()).mean() > 0.98
