"""Canonical coordinates at the ranks whose projection step holds whole rows in
registers (k = 16, 32) and beside them, at row counts around a work-group's
256 rows and with more rows than the largest grid covers at once."""
import numpy as np
import pytest
import torch

import oracle.warmstart_oracle as w
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, to_dev  # noqa: E402


@pytest.mark.parametrize("n,width,k", [(16, 16, 16), (40, 17, 16), (255, 64, 32), (257, 32, 32), (513, 40, 31),
                                       (1100, 64, 16), (263000, 20, 16)])
def test_canonical_matches_oracle(n, width, k):
    Y = np.random.default_rng(n).normal(size=(n, width)) * np.linspace(1.0, 3.0, width)
    Y = Y.astype(np.float32).astype(np.float64)
    Xr, anch_r = w.canonical_coordinates(Y, k, width)
    X = torch.empty(n, width, device=dev())
    anchors = torch.empty(k, dtype=torch.int64, device=dev())
    sym.symnmf_canonical(ctx(), to_dev(Y), k, X, anchors)
    picked = anchors.cpu().tolist()
    if n == width == k:                                   # all residual rows tie: any order of all rows
        assert sorted(picked) == list(range(n))
        return
    assert picked == anch_r.tolist()
    # FP64 work on both sides, stored as float32 (2^-24 relative to each entry)
    assert np.max(np.abs(from_dev(X) - Xr)) <= 1e-7 * max(1.0, np.max(np.abs(Xr)))
