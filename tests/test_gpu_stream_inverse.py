"""ADMM steps whose inverse the stream's launch forms beside its products: every
storage type and column width of the quarter-tile kernel, a size at which its
work-groups fill the card (the inverse then takes one's place at 64 columns),
several steps in a row (each inverse from the Gram of the step before), and a
row panel."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy  # noqa: E402


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,k,steps", [(300, 9, 4), (600, 32, 3), (300, 64, 3), (4100, 50, 1), (2100, 64, 2)])
def test_steps_against_oracle(dtype, n, k, steps):
    c = ctx()
    g = torch.Generator("cuda").manual_seed(n + k)
    X = torch.randn(40, n, generator=g, device=dev()) + torch.randn(40, 1, generator=g, device=dev())
    S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype])
    M = stored_numpy(S)
    H0 = (0.1 + np.random.default_rng(k).random((n, k)) * (np.random.default_rng(k + 1).random((n, k)) < 0.3))
    H0 = H0.astype(np.float32).astype(np.float64)
    p = dict(rho=0.5 * n)                    # of the size of H^T H: a well-conditioned matrix
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=sym.ADMM, **p),
                                 torch.tensor(H0, dtype=torch.float32, device=dev()))
    solver = o.Solver(M, k, o.Params(method=o.ADMM, **p), H0)
    for _ in range(steps):
        sym.symnmf_step(c, S, st)
        solver.step()
    got = from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, device=dev())))
    # products summed in FP32, a few steps: the bound of one step per step
    assert np.max(np.abs(got - solver.H)) <= steps * 2e-4 * max(1.0, np.max(np.abs(solver.H)))


@pytest.mark.parametrize("row0,rows", [(0, 300), (256, 700), (1300, 511)])
def test_panel_equals_rows_of_the_full_step(row0, rows):
    c, n, k = ctx(), 1900, 33
    g = torch.Generator("cuda").manual_seed(row0)
    X = torch.randn(50, n, generator=g, device=dev()) + torch.randn(50, 1, generator=g, device=dev())
    H0 = torch.rand(n, k, generator=g, device=dev())
    p = sym.symnmf_params_default(method=sym.ADMM, rho=500.0)
    out = []
    for kw in (dict(), dict(row0=row0, rows=rows)):
        S = sym.symnmf_build_S(c, X, **kw)
        st = sym.symnmf_state_create(c, S, k, p, H0)
        sym.symnmf_step(c, S, st)
        out.append(from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, device=dev())))[row0:row0 + rows])
    # the same products in another split
    assert np.max(np.abs(out[0] - out[1])) <= 2e-5 * max(1.0, np.max(np.abs(out[0])))
