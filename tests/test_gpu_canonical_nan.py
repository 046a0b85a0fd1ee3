"""Canonical coordinates of a sketch with NaN entries: a column with a NaN takes
no part, and the rows without one get the coordinates they have when that
column is zero; ENUMERIC where the column would have to be taken."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev  # noqa: E402


@pytest.mark.parametrize("n,w,k,bad", [(700, 33, 17, [(3, 32)]), (700, 64, 16, [(3, 40)]), (5000, 64, 32, [(3, 63), (9, 62)]),
                                       (300, 5, 2, [(3, 4)])])
def test_rows_without_a_nan(n, w, k, bad):
    g = torch.Generator("cuda").manual_seed(n + w)
    # columns of falling size, so that the ones with a NaN are not among the k largest
    Y = torch.randn(n, w, generator=g, device=dev()) * (2.0 - torch.arange(w, device=dev()) / w)
    Y[[r for r, _ in bad]] *= 1e-3                       # no anchors among the rows with a NaN
    clean, anchors, got_anchors = Y.clone(), *(torch.empty(k, dtype=torch.int64, device=dev()) for _ in range(2))
    for r, col in bad:
        Y[r, col] = float("nan")
        clean[:, col] = 0.0
    want, got = torch.empty(n, w, device=dev()), torch.empty(n, w, device=dev())
    sym.symnmf_canonical(ctx(), clean, k, want, anchors)
    sym.symnmf_canonical(ctx(), Y, k, got, got_anchors)
    want, got = from_dev(want), from_dev(got)
    rows = np.setdiff1d(np.arange(n), [r for r, _ in bad])
    assert torch.equal(anchors, got_anchors)
    # the same FP64 arithmetic; FP32 output
    assert np.max(np.abs(got[rows] - want[rows])) <= 1e-6 * np.max(np.abs(want[rows]))
    assert np.all(np.isnan(got[[r for r, _ in bad], :k]))


@pytest.mark.parametrize("w,k,col", [(16, 4, 0), (16, 16, 7)])
def test_a_column_that_is_needed(w, k, col):
    Y = torch.randn(400, w, generator=torch.Generator("cuda").manual_seed(w), device=dev())
    Y[3, col] = float("nan")
    with pytest.raises(sym.SymnmfError) as e:
        sym.symnmf_canonical(ctx(), Y, k, torch.empty(400, w, device=dev()))
    assert e.value.code == sym.ENUMERIC
