"""K-means kernels where a work-group's run spans several units: the cluster sums
from column lists against the dense product's (the same order of summation, so
the same bits before the columns are normalised), and an assignment whose last
two slices are one 80-column pass."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, untile  # noqa: E402


def store(n):
    g = torch.Generator("cuda").manual_seed(n)
    X = torch.randn(60, n, generator=g, device=dev()) + torch.randn(60, 1, generator=g, device=dev())
    return sym.symnmf_build_S(ctx(), X), g


def dense(S):
    d = S.desc
    return untile(S.buf[: d.rows_pad * d.ld * 4].view(torch.float32), d.rows_pad, d.ld, 4)[: d.n, : d.n].double()


@pytest.mark.parametrize("n", [9000, 14000])
def test_sums_from_lists_equal_the_dense_product(n):
    S, g = store(n)
    labels = torch.randint(0, 32, (n,), generator=g, device=dev(), dtype=torch.int32)
    C32, C33 = torch.empty(n, 32, device=dev()), torch.empty(n, 33, device=dev())
    sym.symnmf_kmeans_centroids(ctx(), S, labels, 32, C32)     # 32 columns: the dense product
    sym.symnmf_kmeans_centroids(ctx(), S, labels, 33, C33)     # 33, one without members: the lists
    torch.cuda.synchronize()
    assert torch.all(C33[:, 32] == 0)
    # equal sums; the FP64 length of a column may be added in another order, so its
    # multiple may round the other way
    assert torch.all((C32 - C33[:, :32]).abs() <= 2.0 ** -23 * C32.abs())


@pytest.mark.parametrize("n,K", [(14000, 141), (14000, 130), (9000, 200)])
def test_assignment_and_update(n, K):
    S, g = store(n)
    D = dense(S)
    norms = D.norm(dim=1)
    rows = torch.randperm(n, generator=g, device=dev())[:K]
    labels, C = torch.empty(n, dtype=torch.int32, device=dev()), torch.empty(n, K, device=dev())
    tol = 4 * np.sqrt(n) * 2.0 ** -24                          # a random walk of n FP32 roundings, on cosines

    def check(Cref, J):
        cos = (D @ Cref) / norms[:, None]
        got = cos.gather(1, labels.long()[:, None])[:, 0]
        assert torch.all(got >= cos.max(1).values - tol)
        assert abs(J - float((1 - got).sum())) <= tol * n

    st = sym.symnmf_kmeans(ctx(), S, K, labels, init_rows=rows.tolist(), tol=0.0, max_iter=0, allow_notconv=True)
    check(D[:, rows] / norms[rows], st["J0"])
    first = labels.clone()
    st = sym.symnmf_kmeans(ctx(), S, K, labels, init_rows=rows.tolist(), tol=0.0, max_iter=1, C=C, allow_notconv=True)
    W = torch.zeros(n, K, dtype=torch.float64, device=dev())
    W[torch.arange(n, device=dev()), first.long()] = 1.0 / norms
    ref = D @ W
    ref = ref / ref.norm(dim=0)
    assert torch.all((C - ref).abs().max(0).values <= tol * ref.abs().max(0).values)
    check(C.double(), st["J"])
