"""S from very many samples of a few instruments: sample counts at which one
work-group per sample, or per 64 samples in a grid's second dimension, is more
than a launch can hold.  FP64 storage, against FP64 sums in torch: a sum of T
terms in any order is within T 2^-53 of its terms' size, and an entry of S is
made of four such sums."""
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import dev, stored_numpy  # noqa: E402


def built(X, **kw):
    c = sym.symnmf_create(0)
    # scratch that has been used before: NaN wherever the call does not write
    work = torch.full((sym.symnmf_build_S_workspace(X.shape[1], X.shape[0], dtype=sym.S_FP64, **kw),), 255,
                      dtype=torch.uint8, device=dev())
    sym.symnmf_set_workspace(c, work)
    try:
        return torch.from_numpy(stored_numpy(sym.symnmf_build_S(c, X, dtype=sym.S_FP64, **kw)))
    finally:
        sym.symnmf_destroy(c)
        del work
        torch.cuda.empty_cache()         # tens of GB, back to the card


def test_correlation_of_more_than_2_24_samples():
    T = 2 ** 24 + 84
    g = torch.Generator("cuda").manual_seed(3)
    X = torch.randn(T, 2, generator=g, device=dev()) + torch.randn(T, 1, generator=g, device=dev())
    S = built(X)
    D = X.double() - X.double().mean(0)
    ref = float((D[:, 0] * D[:, 1]).sum().abs() / (D[:, 0].norm() * D[:, 1].norm()))
    assert abs(float(S[0, 1]) - ref) <= 4 * T * 2.0 ** -53
    assert float(S[1, 0]) == float(S[0, 1]) and float(S[0, 0]) == 1.0
