"""The quarter-tile stream kernel of small full steps against the one that
larger ones run, and at the edges of its range: one tile, ragged last tiles and
chunks, work-groups whose runs cross tiles, row panels, every storage type and
column width, sizes on both sides of its limits."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_rows, to_dev  # noqa: E402


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,row0,rows,k", [(64, 0, 64, 16), (257, 0, 257, 7), (700, 0, 700, 32), (2100, 0, 2100, 64),
                                           (4100, 0, 4100, 20), (5000, 1300, 300, 33), (30000, 256, 511, 17),
                                           (7000, 0, 7000, 40), (7200, 0, 7200, 64), (8192, 0, 8192, 32),
                                           (8193, 0, 8193, 16), (12300, 0, 12300, 32)])
def test_gradient_of_a_full_step(dtype, n, row0, rows, k):
    c = ctx()
    g = torch.Generator("cuda").manual_seed(n + k)
    X = torch.randn(40, n, generator=g, device=dev()) + torch.randn(40, 1, generator=g, device=dev())
    S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype], row0=row0, rows=rows)
    H0 = torch.rand(n, k, generator=g, device=dev()) * 0.3
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=sym.MU, eps=2.0 ** -23), H0)
    s = sym.symnmf_step(c, S, st)
    G = from_dev(sym.symnmf_state_read(c, st, 6, torch.empty(rows, k, device=dev())))
    H = from_dev(H0)
    own = np.arange(row0, row0 + rows)
    pick = np.unique(np.concatenate([own[[0, -1]], np.random.default_rng(1).choice(own, min(rows, 40))]))
    Sr = stored_rows(S, pick)
    ref = 4.0 * (H[pick] @ (H.T @ H) - Sr @ H)
    # FP32 products and sums over n terms, against the largest term of the difference
    scale = 4.0 * np.max(np.abs(Sr) @ np.abs(H))
    assert np.max(np.abs(G[pick - row0] - ref)) <= 2e-5 * scale
    assert s.full == 1 and np.isfinite(s.f)
