"""pruner_pacm_score in one launch (sets of at most 64 candidates per compute unit) against the three launches of larger sets: the
same bits, at the sizes where a workgroup's share changes, with counts that leave tiles of the branches empty or full."""
import numpy as np
import pytest
import torch

import workloads as w
from test_gpu_parity import P, dev, gpu_pacm  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


def _set(n_d, kind):
    rng = np.random.default_rng(n_d)
    if kind == "none":
        n_stmt, n_blk = np.zeros(n_d, np.int32), np.zeros(n_d, np.int32)
    elif kind == "full":
        n_stmt, n_blk = np.full(n_d, 8, np.int32), np.full(n_d, 8, np.int32)
    else:
        n_stmt, n_blk = rng.integers(0, 9, size=n_d).astype(np.int32), rng.integers(0, 9, size=n_d).astype(np.int32)
    g = torch.Generator(device="cuda")
    g.manual_seed(n_d)
    feat = torch.rand((n_d, 8, 164), generator=g, device="cuda") * 24
    flow = torch.rand((n_d, 8, 23), generator=g, device="cuda") * 24
    return feat, dev(n_stmt), flow, dev(n_blk)


@pytest.mark.parametrize("kind", ["mixed", "none", "full"])
@pytest.mark.parametrize("per_cu", [8, 40, 64])
def test_one_launch_has_the_bits_of_three(P, per_cu, kind):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    gm = gpu_pacm(w.make_pacm_weights(seed=2))
    large = 64 * cus + 1   # the first size that takes three launches
    feat, n_stmt, flow, n_blk = _set(large, kind)
    want = P.pacm_score(feat, n_stmt, flow, n_blk, gm).view(torch.int32)
    for n in (per_cu * cus - 1, per_cu * cus, per_cu * cus + 1, per_cu - 7, 33):
        if n >= large:
            continue
        got = P.pacm_score(feat[:n], n_stmt[:n], flow[:n], n_blk[:n], gm).view(torch.int32)
        assert torch.equal(got, want[:n]), n
