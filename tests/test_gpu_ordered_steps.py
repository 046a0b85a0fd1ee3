"""Several steps in a row at ranks other than 16, 32 and 64 with the methods that
sum by increasing column: from the second step on the images of H are the FP32
ones that the update kernels write, on BF16 and FP8 storage too, those of 2 H
for block steps among them, and a state moves between storages.  Every step's
gradient against FP64 at the iterate it was taken at (a stale or wrong image is
off by the step's own size, far above the FP32 bound); sampled steps against
the oracle.  And ADMM steps of row panels small enough that the stream's launch
forms the inverse."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy, to_dev  # noqa: E402


def returns(n, seed=0):
    g = torch.Generator("cuda").manual_seed(n + seed)
    return torch.randn(40, n, generator=g, device=dev()) + torch.randn(40, 1, generator=g, device=dev())


def check_steps(c, st, S, k, steps, row0=0):
    n, rows, M = S.desc.n, S.desc.rows, stored_numpy(S)
    for _ in range(steps):
        H = from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, device=dev())))
        sym.symnmf_step(c, S, st, want_stats=False)
        G = from_dev(sym.symnmf_state_read(c, st, 6, torch.empty(rows, k, device=dev())))
        own = H[row0:row0 + rows]
        # FP32 products and sums over n terms, against the largest term of the difference
        scale = 4.0 * max(np.max(np.abs(M) @ np.abs(H)), np.max(np.abs(own) @ (np.abs(H).T @ np.abs(H))))
        assert np.max(np.abs(G - 4.0 * (own @ (H.T @ H) - M @ H))) <= 2e-6 * scale


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,row0,rows,k,method", [(1100, 0, 1100, 20, sym.ADMM), (1300, 0, 1300, 50, sym.ADMM),
                                                  (700, 0, 700, 5, sym.ADAGRAD), (1500, 320, 500, 33, sym.ADAM),
                                                  (1500, 130, 301, 17, sym.ADMM)])
def test_gradients_of_consecutive_steps(dtype, n, row0, rows, k, method):
    c = ctx()
    S = sym.symnmf_build_S(c, returns(n), dtype=sym.DTYPES[dtype], row0=row0, rows=rows)
    H0 = torch.rand(n, k, generator=torch.Generator("cuda").manual_seed(k), device=dev()) * 0.3
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=method, eta=0.05, rho=50.0), H0)
    check_steps(c, st, S, k, 4, row0)


@pytest.mark.parametrize("n,k,method", [(1200, 20, sym.ADMM), (600, 37, sym.ADAGRAD), (900, 50, sym.ADMM)])
def test_gradients_across_storages(n, k, method):
    c, X = ctx(), returns(n)
    H0 = torch.rand(n, k, generator=torch.Generator("cuda").manual_seed(k), device=dev()) * 0.3
    Ss = [sym.symnmf_build_S(c, X, dtype=sym.DTYPES[d]) for d in ("fp32", "bf16", "fp8", "fp32")]
    st = sym.symnmf_state_create(c, Ss[0], k, sym.symnmf_params_default(method=method, eta=0.05, rho=50.0), H0)
    for i, S in enumerate(Ss):
        if i:
            sym.symnmf_state_rebind(c, st, S)
        check_steps(c, st, S, k, 2)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("method,k", [("block", 20), ("block", 33), ("row", 5)])
def test_sampled_steps_match_oracle(dtype, method, k):
    Snp = o.abs_corr(synth.c1_instance(5, T=1500, n=1300, groups=7).X.numpy())
    kw = dict(eta=0.05, eps=1e-3, block_rows=256, snapshot_s=5, seed=11)
    m, r = (sym.BLOCK_SVRG, o.BLOCK_SVRG) if method == "block" else (sym.ROW_SVRG, o.ROW_SVRG)
    kw.update(dict(phi0=0.4) if method == "block" else dict(row_frac=0.4))
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(Snp, torch.float64), dtype=sym.DTYPES[dtype])
    H0 = o.init_H(Snp.mean(), 1300, k, 3, as_float32=True)
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=m, **kw), to_dev(H0))
    solver = o.Solver(stored_numpy(S), k, o.Params(method=r, **kw), H0)
    for _ in range(8):
        sym.symnmf_step(c, S, st, want_stats=False)
        solver.step()
    got = from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(1300, k, device=dev())))
    assert np.max(np.abs(got - solver.H)) <= 1e-4            # the bound of these runs on FP32 storage


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("row0,rows,k", [(0, 300, 33), (256, 513, 64), (130, 301, 9), (960, 64, 32)])
def test_small_admm_panel_equals_rows_of_the_full_step(dtype, row0, rows, k):
    c, n = ctx(), 1024
    X, H0 = returns(n, row0), torch.rand(n, k, generator=torch.Generator("cuda").manual_seed(row0), device=dev())
    p = sym.symnmf_params_default(method=sym.ADMM, rho=500.0)
    out = []
    for kw in (dict(), dict(row0=row0, rows=rows)):
        S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype], fp8_panel_rows=1, **kw)   # scales of a row: the same in both
        st = sym.symnmf_state_create(c, S, k, p, H0)
        sym.symnmf_step(c, S, st)
        out.append(from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, device=dev())))[row0:row0 + rows])
    # the same products in another split
    assert np.max(np.abs(out[0] - out[1])) <= 2e-5 * max(1.0, np.max(np.abs(out[0])))
