"""The stream kernel that sums by increasing column, one rounding a product: the
gradients it gives against those sums formed one by one, and against 64 bits at
ragged tiles, runs of several units, row panels and every storage type."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy, stored_rows  # noqa: E402


def one_step(dtype, n, row0, rows, k, method):
    c = ctx()
    g = torch.Generator("cuda").manual_seed(n + k)
    X = torch.randn(40, n, generator=g, device=dev()) + torch.randn(40, 1, generator=g, device=dev())
    S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype], row0=row0, rows=rows)
    H0 = torch.rand(n, k, generator=g, device=dev()) * 0.3
    st = sym.symnmf_state_create(c, S, k, sym.symnmf_params_default(method=method), H0)
    s = sym.symnmf_step(c, S, st)
    G = sym.symnmf_state_read(c, st, 6, torch.empty(rows, k, device=dev()))
    return S, from_dev(H0), G.cpu().numpy(), s


def chain(A, B):
    """A B with FP32 multiply-adds by increasing inner index (80-bit products and sums, rounded each time)."""
    acc = np.zeros((A.shape[0], B.shape[1]), np.float32)
    A, B = A.astype(np.longdouble), B.astype(np.longdouble)
    for j in range(A.shape[1]):
        acc = (acc + A[:, j:j + 1] * B[j]).astype(np.float32)
    return acc


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("n,k", [(200, 5), (257, 20), (600, 50)])
def test_order_of_the_products(dtype, n, k):
    # at most nine units, one a work-group: a partial per 256 columns, added by increasing column
    S, H, G, _ = one_step(dtype, n, 0, n, k, sym.ADAGRAD)
    M = stored_numpy(S)
    sw = np.zeros((n, k), np.float32)
    for c0 in range(0, n, 256):
        sw = sw + chain(M[:, c0:c0 + 256], H[c0:c0 + 256])
    gram = (H.T @ H).astype(np.float32)
    assert np.array_equal(G, np.float32(4) * (chain(H, gram) - sw))


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,row0,rows,k,method", [(1, 0, 1, 1, sym.ADAGRAD), (255, 0, 255, 17, sym.ADAGRAD),
                                                  (1025, 0, 1025, 15, sym.ADMM), (1024, 0, 1024, 15, sym.ADMM),
                                                  (2100, 0, 2100, 20, sym.ADMM), (6100, 0, 6100, 33, sym.ADMM),
                                                  (8200, 0, 8200, 63, sym.ADAGRAD), (9000, 1300, 300, 31, sym.ADAGRAD)])
def test_gradient_against_64_bits(dtype, n, row0, rows, k, method):
    S, H, G, s = one_step(dtype, n, row0, rows, k, method)
    own = np.arange(row0, row0 + rows)
    pick = np.unique(np.concatenate([own[[0, -1]], np.random.default_rng(1).choice(own, min(rows, 40))]))
    Sr = stored_rows(S, pick)
    ref = 4.0 * (H[pick] @ (H.T @ H) - Sr @ H)
    # FP32 products and sums over n terms, against the largest term of the difference
    scale = 4.0 * np.max(np.abs(Sr) @ np.abs(H))
    assert np.max(np.abs(G[pick - row0] - ref)) <= 2e-5 * scale
    assert s.full == 1 and np.isfinite(s.f)
