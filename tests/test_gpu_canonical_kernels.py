"""Canonical coordinates where their kernels change form: odd widths (the
rotation order has a bye), one column, all columns, row counts around the 64-
and 256-row blocks, several work-groups in the anchor search."""
import numpy as np
import pytest
import torch

import oracle.warmstart_oracle as w
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, to_dev  # noqa: E402


@pytest.mark.parametrize("n,width,k", [(1, 1, 1), (5, 3, 2), (64, 64, 64), (65, 33, 20), (257, 63, 63), (256, 16, 1),
                                       (1025, 64, 33)])
def test_canonical_matches_oracle(n, width, k):
    Y = np.random.default_rng(n).normal(size=(n, width)).astype(np.float32).astype(np.float64)
    Xr, anch_r = w.canonical_coordinates(Y, k, width)
    X = torch.empty(n, width, device=dev())
    anchors = torch.empty(k, dtype=torch.int64, device=dev())
    sym.symnmf_canonical(ctx(), to_dev(Y), k, X, anchors)
    Xg = from_dev(X)
    if n == k:
        # Z is orthogonal: every residual row is as long as the next, so rounding alone
        # orders the anchors; they are all the rows, and the coordinates their unit rows
        picked = anchors.cpu().tolist()
        assert sorted(picked) == list(range(n))
        assert np.max(np.abs(Xg[picked, :k] - np.eye(k))) <= 1e-7
        return
    assert anchors.cpu().tolist() == anch_r.tolist()
    assert np.all(Xg[:, k:] == 0.0)
    # FP64 work on both sides, stored as float32 (2^-24 relative to each entry)
    assert np.max(np.abs(Xg - Xr)) <= 1e-7 * max(1.0, np.max(np.abs(Xr)))
