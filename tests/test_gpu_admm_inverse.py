"""The ADMM step's k x k inverse at the edges of its register blocks, through
one step of an FP64 state (exact to FP64 rounding) and of an FP32 one."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, to_dev  # noqa: E402


@pytest.mark.parametrize("dtype,k", [("fp64", 1), ("fp64", 2), ("fp64", 16), ("fp64", 17), ("fp64", 31), ("fp64", 32),
                                     ("fp32", 1), ("fp32", 16), ("fp32", 17), ("fp32", 33), ("fp32", 62), ("fp32", 63),
                                     ("fp32", 64)])
@pytest.mark.parametrize("rho", [0.5, 500.0])
def test_admm_step(dtype, k, rho):
    n, f64 = 300, dtype == "fp64"
    Snp = o.abs_corr(synth.c1_instance(6, T=900, n=n, groups=6).X.numpy())
    if not f64:
        Snp = Snp.astype(np.float32).astype(np.float64)
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(Snp, torch.float64), dtype=sym.DTYPES[dtype])
    # a factor whose Gram is well conditioned, so that the step, not the inverse's
    # condition, sets the error
    H0 = 0.1 + np.random.default_rng(k).random((n, k)) * (np.random.default_rng(k + 1).random((n, k)) < 0.3)
    H0 = H0 if f64 else H0.astype(np.float32).astype(np.float64)
    tdt = torch.float64 if f64 else torch.float32
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=sym.ADMM, rho=rho), to_dev(H0, tdt))
    sym.symnmf_step(c, S, st)
    got = from_dev(sym.symnmf_state_read(c, st, 0, torch.empty(n, k, dtype=tdt, device=dev())))
    solver = o.Solver(Snp, k, o.Params(method=o.ADMM, rho=rho), H0)
    solver.step()
    # FP64: rounding times the condition of 2 W^T W + rho I (below 1e4); FP32: products summed in FP32
    assert np.max(np.abs(got - solver.H)) <= (1e-11 if f64 else 2e-4) * max(1.0, np.max(np.abs(solver.H)))
