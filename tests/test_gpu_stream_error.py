"""The streams of MU and small ADMM steps are no further from 64 bits than the
kernels of the other methods, whose order of summation these steps had
before: the gradient at a given H, against FP64, of an MU step and of an AdaGrad
step, at the sizes with the longest runs of units and at single tiles of few
columns.  Both errors are sums over all entries (and seeds), so the comparison
needs no slack."""
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, stored_numpy, untile  # noqa: E402


def dense(S):
    d = S.desc
    if d.dtype == sym.S_FP32:
        return untile(S.buf[: d.rows_pad * d.ld * 4].view(torch.float32), d.rows_pad, d.ld, 4)[: d.n, : d.n].double()
    return torch.from_numpy(stored_numpy(S)).to(dev())


def errors(dtype, n, k, seeds, methods):
    c, err = ctx(), [0.0] * len(methods)
    for seed in range(seeds):
        g = torch.Generator("cuda").manual_seed(1000 * seed + n + k)
        X = torch.randn(80, n, generator=g, device=dev()) + torch.randn(80, 1, generator=g, device=dev())
        S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype])
        H0 = 0.3 * torch.rand(n, k, generator=g, device=dev()) * (torch.rand(n, k, generator=g, device=dev()) < 0.6)
        H = H0.double()
        ref = 4.0 * (H @ (H.T @ H) - dense(S) @ H)
        for i, method in enumerate(methods):
            st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=method), H0)
            sym.symnmf_step(c, S, st, want_stats=False)
            G = sym.symnmf_state_read(c, st, 6, torch.empty(n, k, device=dev()))
            err[i] += float(((G.double() - ref) ** 2).sum() / (ref ** 2).sum()) / seeds
    print(f"{dtype} n={n} k={k}: " + "  ".join(f"{e ** 0.5:.3e}" for e in err))
    return err


@pytest.mark.parametrize("dtype,n,k", [("fp32", 5900, 64), ("fp32", 8200, 20), ("fp32", 8200, 32), ("fp32", 10000, 17),
                                       ("fp32", 12200, 32), ("bf16", 8100, 20), ("fp8", 8100, 31),
                                       ("fp32", 13000, 5), ("fp32", 18000, 20), ("fp32", 18000, 50)])
def test_long_runs(dtype, n, k):
    mu, before = errors(dtype, n, k, 1, (sym.MU, sym.ADAGRAD))
    assert mu <= before


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("n,k", [(20, 2), (20, 13), (37, 1), (37, 20), (70, 40)])
def test_few_columns(dtype, n, k):
    mu, admm, before = errors(dtype, n, k, 30, (sym.MU, sym.ADMM, sym.ADAGRAD))
    assert mu <= before and admm <= before
