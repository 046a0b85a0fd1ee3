"""The training step's kernels at the edges of their tiles: ranks that fill a
16-column block, leave a remainder or are a single column, row counts around
the 64- and 128-row blocks, a hidden width that is no multiple of 64; and a
step whose loss cannot be formed, which must leave the network as it was."""
import numpy as np
import pytest
import torch

import oracle.warmstart_oracle as w
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, to_dev  # noqa: E402
from test_gpu_warmstart import _flat, _params32, _unflat  # noqa: E402


@pytest.mark.parametrize("k,m,width,hidden,residual,kind", [
    (1, 63, 20, 36, False, 0), (5, 129, 64, 256, True, 1), (16, 64, 33, 100, True, 0), (17, 1025, 64, 256, False, 1),
    (33, 128, 64, 72, True, 1), (64, 577, 64, 256, True, 1), (64, 130, 64, 64, False, 0)])
def test_gradient_matches_oracle(k, m, width, hidden, residual, kind):
    P = _params32(k, seed=k + m, width=width, hidden=hidden)
    g = np.random.default_rng(m)
    Xin = g.normal(size=(m, width)).astype(np.float32).astype(np.float64)
    B = g.random((m, k)).astype(np.float32).astype(np.float64)
    A, cache = w.forward(P, Xin, residual)
    L_ref, dA = (w.gram_loss if kind == 0 else w.gram_cos_loss)(A, B)
    G_ref = w.backward(P, cache, dA)
    c = ctx()
    net = sym.symnmf_mlp_create(c, width, hidden, k, to_dev(_flat(P)))
    sym.symnmf_mlp_set_output(c, net, residual)
    L = sym.symnmf_mlp_train_step(c, net, to_dev(Xin), to_dev(B), loss_kind=kind)
    assert L == pytest.approx(L_ref, rel=1e-5, abs=1e-6)
    G = _unflat(from_dev(sym.symnmf_mlp_read(c, net, "grad", torch.empty(net.count, device=dev()))), width, hidden, k)
    for name in G_ref:
        # FP32 products and sums behind every entry; the repository's bound for a training step
        assert np.max(np.abs(G[name] - G_ref[name])) <= 1e-3 * np.max(np.abs(G_ref[name])), name


@pytest.mark.parametrize("bad,code", [("target", sym.EINVAL), ("output", sym.ENUMERIC), ("nan", sym.ENUMERIC)])
def test_refused_step_changes_nothing(bad, code):
    k, m, width, hidden = 6, 200, 64, 64
    P = _params32(k, seed=3, width=width, hidden=hidden)
    g = np.random.default_rng(5)
    good_X, good_B = g.random((m, width)), g.random((m, k))
    c = ctx()
    if bad == "output":                     # a residual network whose output is max(X, 0) = 0
        P["W3"][:] = 0.0
        P["b3"][:] = 0.0
        good_X = -good_X
    net = sym.symnmf_mlp_create(c, width, hidden, k, to_dev(_flat(P)))
    sym.symnmf_mlp_set_output(c, net, bad == "output")
    if bad != "output":
        sym.symnmf_mlp_train_step(c, net, to_dev(good_X), to_dev(good_B), loss_kind=1)
    before = [from_dev(sym.symnmf_mlp_read(c, net, which, torch.empty(net.count, device=dev())))
              for which in ("params", "grad", "m", "v")]
    X, B = good_X.copy(), good_B.copy()
    if bad == "target":
        B[:] = 0.0
    if bad == "nan":
        B[7, 2] = np.nan
        code = sym.EINVAL                   # B^T B is not finite
    with pytest.raises(sym.SymnmfError) as e:
        sym.symnmf_mlp_train_step(c, net, to_dev(X), to_dev(B), loss_kind=1)
    assert e.value.code == code
    if bad == "nan":
        X[3, 1] = np.nan
        with pytest.raises(sym.SymnmfError) as e:
            sym.symnmf_mlp_train_step(c, net, to_dev(X), to_dev(good_B), loss_kind=0)
        assert e.value.code == sym.ENUMERIC
    for which, ref in zip(("params", "grad", "m", "v"), before):
        got = from_dev(sym.symnmf_mlp_read(c, net, which, torch.empty(net.count, device=dev())))
        assert np.array_equal(got, ref), which


@pytest.mark.parametrize("n,k", [(64, 1), (129, 3), (300, 17), (1000, 64)])
def test_subspace_error_of_rotated_factors_is_zero(n, k):
    """The blocked X^T Y products through a value known exactly: the column
    span of A M equals A's for an invertible M."""
    g = np.random.default_rng(k)
    A = g.normal(size=(n, k))
    B = A @ (g.normal(size=(k, k)) + 3.0 * np.eye(k))
    got = sym.symnmf_subspace_error(ctx(), to_dev(A), to_dev(B))
    # A M is rounded to float32: 2^-24 relative times the condition of M (below 1e3)
    assert got < 1e-4
