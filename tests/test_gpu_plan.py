"""Plans of sampled steps where the plan kernel changes form: one block, one
more than a round of its 256 threads in blocks, tiles and chunks, block sizes of
several tiles, principal and independent sets."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_rows, to_dev  # noqa: E402


@pytest.mark.parametrize("method", [sym.ROW_SVRG, sym.BLOCK_SVRG])
@pytest.mark.parametrize("n,block_rows,indep", [(300, 512, 1), (1300, 512, 1), (1300, 256, 0), (66000, 256, 1),
                                                (66000, 1024, 0)])
def test_sampled_gradient(method, n, block_rows, indep):
    k, c = 16, ctx()
    X = torch.randn(24, n, generator=torch.Generator("cuda").manual_seed(n), device=dev())
    X += torch.randn(24, 1, generator=torch.Generator("cuda").manual_seed(3), device=dev())
    S = sym.symnmf_build_S(c, X, dtype=sym.S_BF16)
    frac = dict(row_frac=0.37) if method == sym.ROW_SVRG else dict(phi0=0.2)
    p = sym.symnmf_params_default(method=method, eta=0.01, eps=1e-3, block_rows=block_rows, snapshot_s=10, seed=5,
                                  independent_blocks=indep, **frac)
    H0 = torch.rand(n, k, generator=torch.Generator("cuda").manual_seed(9), device=dev()) * 0.1
    st = sym.symnmf_state_create(c, S, k, p, H0)
    sym.symnmf_step(c, S, st, want_stats=False)                       # t = 0: the snapshot
    H = from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, device=dev())))
    mu = from_dev(sym.symnmf_state_read(c, st, 5, torch.empty(n, k, device=dev())))
    sym.symnmf_step(c, S, st, want_stats=False)                       # t = 1: sampled
    G = from_dev(sym.symnmf_state_read(c, st, 6, torch.empty(n, k, device=dev())))
    nb = -(-n // block_rows)
    m = min(nb, int(np.ceil((0.37 if method == sym.ROW_SVRG else np.sqrt(0.2)) * nb)))
    block_of = np.arange(n) // block_rows
    inI = np.isin(block_of, sym.symnmf_sample_blocks(5, 1, 0, nb, m))
    inJ = inI if not indep else np.isin(block_of, sym.symnmf_sample_blocks(5, 1, 1, nb, m))
    if method == sym.ROW_SVRG:
        inJ = np.zeros(n, bool)
    out = ~(inI | inJ)
    assert np.array_equal(G[out], mu[out])                            # the others keep the snapshot gradient
    rng = np.random.default_rng(1)
    for sel in (inI & ~inJ, inJ & ~inI, inI & inJ):
        rows = np.nonzero(sel)[0]
        if rows.size == 0:
            continue
        rows = np.unique(np.concatenate([rows[[0, -1]], rng.choice(rows, 6)]))
        Sr = stored_rows(S, rows)
        if method == sym.ROW_SVRG:
            ref = 4.0 * (H[rows] @ (H.T @ H) - Sr @ H)
        else:
            ref = np.zeros((rows.size, k))
            if sel[rows[0]] and inI[rows[0]]:
                ref += 2.0 * (H[rows] @ (H[inJ].T @ H[inJ]) - Sr[:, inJ] @ H[inJ])
            if inJ[rows[0]]:
                ref += 2.0 * (H[rows] @ (H[inI].T @ H[inI]) - Sr[:, inI] @ H[inI])
        # FP32 products and sums over up to 66000 terms
        assert np.max(np.abs(G[rows] - ref)) <= 1e-4 * np.max(np.abs(ref))
