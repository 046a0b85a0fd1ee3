"""K-means at the edges of its kernels: the cluster sums of FP32 storage (lists
of a chunk's columns, passes of 192 clusters, runs of units of a tile pair), the
last, narrower slice of a product (together with the one before it where it has
at most 16 columns), and the assignment's four lanes to a row.

Oracle: FP64 on the stored S.  A centroid entry is a sum of at most n FP32 terms
of one sign times one factor: its error is a random walk, at most
4 sqrt(n) 2^-24 of the sum for the sizes here, the same relative to the
column's largest entry after normalising.  An assignment's product has the same
bound on its cosine; the choice must be within that of the best one."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy  # noqa: E402


def _store(n, dtype, seed=0):
    g = torch.Generator("cuda").manual_seed(seed + n)
    X = torch.randn(60, n, generator=g, device=dev()) + torch.randn(60, 1, generator=g, device=dev())
    S = sym.symnmf_build_S(ctx(), X, kind=sym.ABS_CORR, dtype=sym.DTYPES[dtype])
    M = stored_numpy(S)
    return S, M, np.sqrt((M * M).sum(1))


def _labels(n, K, kind):
    r = np.random.default_rng(n + K)
    if kind == "one":                   # every column in one cluster: the longest list of a block
        return np.full(n, K - 1)
    if kind == "blocks":                # whole chunks in one 16-cluster block
        return (np.arange(n) // 256 * 16 + r.integers(0, 16, n)) % K
    if kind == "few":                   # empty clusters, most columns in none
        lab = np.full(n, -1)
        lab[r.choice(n, K // 2, replace=False)] = r.permutation(K)[:K // 2]
        return lab
    return r.integers(0, K, n)


@pytest.mark.parametrize("n,K", [(33, 33), (256, 64), (257, 65), (600, 128), (1100, 129), (1100, 192), (900, 193),
                                 (2600, 400), (5000, 141)])
@pytest.mark.parametrize("kind", ["random", "one", "blocks", "few"])
def test_centroids(n, K, kind):
    S, M, norms = _store(n, "fp32")
    lab = _labels(n, K, kind)
    prev = torch.rand(n, K, generator=torch.Generator("cuda").manual_seed(K), device=dev())
    C = torch.empty(n, K, device=dev())
    sym.symnmf_kmeans_centroids(ctx(), S, torch.tensor(lab, dtype=torch.int32, device=dev()), K, C, C_prev=prev)
    W = np.zeros((n, K))
    own = lab >= 0
    W[np.nonzero(own)[0], lab[own]] = 1.0 / norms[own]
    ref = M @ W
    length = np.sqrt((ref * ref).sum(0))
    some = length > 0
    ref = np.where(some, ref / np.where(some, length, 1.0), from_dev(prev))
    err = np.max(np.abs(from_dev(C) - ref), axis=0)
    assert np.all(err[~some] == 0)
    assert np.all(err[some] <= 4 * np.sqrt(n) * 2.0 ** -24 * np.max(np.abs(ref[:, some]), axis=0))


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,K", [(70, 65), (300, 80), (300, 81), (513, 100), (600, 129), (1100, 141), (1100, 190),
                                 (2900, 200), (1300, 3), (700, 1)])
def test_assignment(dtype, n, K):
    S, M, norms = _store(n, dtype)
    g = torch.Generator("cuda").manual_seed(K)
    C = torch.rand(n, K, generator=g, device=dev())
    C[:, K // 2] = C[:, 0]              # equal products: the lower index
    C /= C.norm(dim=0)
    C[:, K // 2] = C[:, 0]
    labels = torch.empty(n, dtype=torch.int32, device=dev())
    best = torch.empty(n, device=dev())
    J = sym.symnmf_kmeans_assign(ctx(), S, C, labels, best)
    cos = (M / norms[:, None]) @ from_dev(C).astype(np.float64)
    lab = from_dev(labels).astype(int)
    tol = 4 * np.sqrt(n) * 2.0 ** -24
    got = cos[np.arange(n), lab]
    assert np.all(got >= cos.max(1) - tol)
    assert K < 2 or not np.any(lab == K // 2)
    assert np.max(np.abs(from_dev(best) - got)) <= tol
    assert abs(float(J) - np.sum(1 - got)) <= tol * n
