"""Ranks and widths that leave columns of the matrix-core stream's 16-column
blocks empty: one column, one more or less than a block, odd sizes, for full,
sampled and row-panel steps, the objective and the sketch, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as o
import oracle.warmstart_oracle as w
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy, to_dev  # noqa: E402

N = 700


@pytest.fixture(scope="module")
def S700():
    return o.abs_corr(synth.c1_instance(4, T=1500, n=N, groups=7).X.numpy())


def _read(c, st, which, k, rows=N):
    return from_dev(sym.symnmf_state_read(c, st, which, torch.empty(rows, k, device=dev())))


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("k", [1, 2, 15, 17, 20, 31, 33, 47, 63])
def test_steps_match_oracle(S700, dtype, k):
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(S700, torch.float64), dtype=sym.DTYPES[dtype], fp8_panel_rows=128)
    Sq = stored_numpy(S)
    H0 = o.init_H(S700.mean(), N, k, 3, as_float32=True)
    for method, rule in ((sym.ADMM, o.ADMM), (sym.MU, o.MU)):
        kw = dict(rho=50.0) if method == sym.ADMM else dict(eps=2.0 ** -23)
        st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=method, **kw), to_dev(H0))
        solver = o.Solver(Sq, k, o.Params(method=rule, **kw), H0)
        for _ in range(3):
            s, r = sym.symnmf_step(c, S, st), solver.step()
            # FP32 products and sums over 700 terms, as for the ranks 16, 32 and 64
            assert s.f == pytest.approx(r.f, rel=2e-5)
        assert np.max(np.abs(_read(c, st, 0, k) - solver.H)) <= 2e-5 * max(1.0, np.max(np.abs(solver.H)))


@pytest.mark.parametrize("method,k", [("block", 20), ("block", 33), ("row", 5)])
def test_sampled_steps_match_oracle(method, k):
    Snp = o.abs_corr(synth.c1_instance(5, T=1500, n=1300, groups=7).X.numpy())
    kw = dict(eta=0.05, eps=1e-3, block_rows=256, snapshot_s=5, seed=11)
    m, r = (sym.BLOCK_SVRG, o.BLOCK_SVRG) if method == "block" else (sym.ROW_SVRG, o.ROW_SVRG)
    kw.update(dict(phi0=0.4) if method == "block" else dict(row_frac=0.4))
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(Snp, torch.float64), dtype=sym.S_FP32)
    H0 = o.init_H(Snp.mean(), 1300, k, 3, as_float32=True)
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=m, **kw), to_dev(H0))
    solver = o.Solver(stored_numpy(S), k, o.Params(method=r, **kw), H0)
    for t in range(8):
        sym.symnmf_step(c, S, st, want_stats=False)
        solver.step()
    assert np.max(np.abs(_read(c, st, 0, k, 1300) - solver.H)) <= 1e-4


def test_panel_and_rebind_at_an_odd_rank(S700):
    k, row0, rows = 21, 130, 301
    c = ctx()
    H0 = o.init_H(S700.mean(), N, k, 3, as_float32=True)
    hi = sym.symnmf_S_load(c, to_dev(S700[row0:row0 + rows], torch.float64), dtype=sym.S_FP32, row0=row0)
    lo = sym.symnmf_S_load(c, to_dev(S700[row0:row0 + rows], torch.float64), dtype=sym.S_FP8, row0=row0)
    st = sym.symnmf_state_create(c, lo, k, sym.symnmf_params_default(method=sym.MU, eps=2.0 ** -23), to_dev(H0))
    sym.symnmf_state_rebind(c, st, hi)
    sym.symnmf_step(c, hi, st, want_stats=False)
    H1 = _read(c, st, 0, k)
    SH, HG = S700[row0:row0 + rows] @ H0, H0[row0:row0 + rows] @ (H0.T @ H0)
    ref = H0.copy()
    ref[row0:row0 + rows] = 0.5 * H0[row0:row0 + rows] * (1.0 + SH / (HG + 2.0 ** -23))
    assert np.max(np.abs(H1 - ref)) <= 2e-5 * np.max(np.abs(ref))
    assert np.array_equal(np.delete(H1, slice(row0, row0 + rows), 0), np.delete(H0, slice(row0, row0 + rows), 0))


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 33, 64])
@pytest.mark.parametrize("f64", [False, True])
def test_objective_matches_oracle(S700, dtype, k, f64):
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(S700, torch.float64), dtype=sym.DTYPES[dtype], fp8_panel_rows=128)
    Sq = stored_numpy(S)
    H = o.init_H(S700.mean(), N, k, 9, as_float32=True)
    f, E = sym.symnmf_objective(c, S, to_dev(H, torch.float64 if f64 else torch.float32), k)
    fro2 = (Sq * Sq).sum()
    ref = o.objective_trace(Sq, H)
    # FP64 H: FP64 products; FP32 H: FP32 sums of at most 256 terms, FP64 across them
    assert abs(f - ref) <= (1e-10 if f64 else 1e-6) * fro2
    assert E == pytest.approx(f / fro2, rel=1e-9)


@pytest.mark.parametrize("width", [1, 10, 33, 63])
def test_sketch_at_odd_widths(S700, width):
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(S700, torch.float64), dtype=sym.S_BF16)
    Y = torch.empty(N, width, device=dev())
    sym.symnmf_sketch(c, S, 17, width, Y)
    Sq, Om = stored_numpy(S), w.omega(17, N, width)
    assert np.all(np.abs(from_dev(Y) - Sq @ Om) <= 2e-5 * (np.abs(Sq) @ np.abs(Om)) + 1e-6)
