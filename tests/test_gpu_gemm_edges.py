"""The network's matrix products at the edges of their vectors and slabs: widths,
hidden sizes and ranks that are no multiple of 4 (rows that start at any entry,
bf16 weights at any two bytes), of 32 or of 64, single rows, row counts around a
64-row tile and around the split of a weight gradient over its rows.

FP32 products and sums of at most 300 terms behind an output (4 sqrt(300) 2^-24
per layer, three layers, against the largest output) and of at most 1100 rows
behind a gradient."""
import numpy as np
import pytest
import torch

import oracle.warmstart_oracle as w
import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, to_dev  # noqa: E402
from test_gpu_warmstart import _flat, _params32, _unflat  # noqa: E402

TOL = 3 * 4 * np.sqrt(300.0) * 2.0 ** -24


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,width,hidden,k", [(1, 1, 1, 1), (63, 19, 37, 5), (64, 33, 66, 31), (65, 7, 129, 3),
                                              (200, 64, 300, 64), (1030, 62, 255, 17)])
def test_forward_and_gradient(m, width, hidden, k, residual):
    P = _params32(k, seed=m + k, width=width, hidden=hidden)
    g = np.random.default_rng(m)
    Xin = g.normal(size=(m, width)).astype(np.float32).astype(np.float64)
    B = (0.1 + g.random((m, k))).astype(np.float32).astype(np.float64)
    c = ctx()
    net = sym.symnmf_mlp_create(c, width, hidden, k, to_dev(_flat(P)))
    sym.symnmf_mlp_set_output(c, net, residual)
    A, cache = w.forward(P, Xin, residual)
    Pb = dict(P, **{n: torch.tensor(P[n]).to(torch.bfloat16).double().numpy() for n in ("W1", "W2", "W3")})
    for bf16, ref in ((False, A), (True, w.forward(Pb, Xin, residual)[0])):
        out = from_dev(sym.symnmf_mlp_forward(c, net, to_dev(Xin), torch.empty(m, k, device=dev()), bf16_weights=bf16))
        assert np.max(np.abs(out - ref)) <= TOL * max(1.0, np.max(np.abs(cache["z3"])))
    if np.max(np.abs(A)) == 0.0:
        return
    L_ref, dA = w.gram_loss(A, B)
    G_ref = w.backward(P, cache, dA)
    L = sym.symnmf_mlp_train_step(c, net, to_dev(Xin), to_dev(B), loss_kind=0)
    assert L == pytest.approx(L_ref, rel=1e-5, abs=1e-6)
    G = _unflat(from_dev(sym.symnmf_mlp_read(c, net, "grad", torch.empty(net.count, device=dev()))), width, hidden, k)
    for name in G_ref:
        # the repository's bound for a training step
        assert np.max(np.abs(G[name] - G_ref[name])) <= 1e-3 * np.max(np.abs(G_ref[name])), name
