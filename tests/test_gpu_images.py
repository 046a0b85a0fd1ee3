"""The images of H that the update kernels leave for the next step: after some
steps, a fresh state created from the iterate takes the next step bit for bit
(its images come from the image kernel), for every storage type, padded ranks,
full matrices and row panels that start on and off a multiple of 64."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, to_dev  # noqa: E402

N = 1000


@pytest.fixture(scope="module")
def S1000():
    return o.abs_corr(synth.c1_instance(7, T=1200, n=N, groups=6).X.numpy())


@pytest.mark.parametrize("dtype,k", [("fp32", 16), ("fp32", 21), ("fp32", 64), ("bf16", 5), ("bf16", 32), ("bf16", 50),
                                     ("fp8", 16), ("fp8", 30), ("fp8", 64)])
@pytest.mark.parametrize("row0,rows", [(0, 1000), (64, 300), (192, 65), (130, 301), (700, 300), (960, 40)])
def test_next_step_equals_a_fresh_state(S1000, dtype, k, row0, rows):
    c = ctx()
    S = sym.symnmf_S_load(c, to_dev(S1000[row0:row0 + rows], torch.float64), dtype=sym.DTYPES[dtype], row0=row0)
    p = sym.symnmf_params_default(method=sym.MU, eps=2.0 ** -23)          # the iterate is the whole state
    st = sym.symnmf_state_create(c, S, k, p, to_dev(o.init_H(0.1, N, k, 3, as_float32=True)))
    H = torch.empty(N, k, device=dev())
    for _ in range(3):
        sym.symnmf_step(c, S, st, want_stats=False)
        sym.symnmf_state_read(c, st, 0, H)
        fresh = sym.symnmf_state_create(c, S, k, p, H)
        sym.symnmf_step(c, S, fresh, want_stats=False)
        want = sym.symnmf_state_read(c, fresh, 6, torch.empty(rows, k, device=dev()))
    sym.symnmf_step(c, S, st, want_stats=False)
    got = sym.symnmf_state_read(c, st, 6, torch.empty(rows, k, device=dev()))
    torch.cuda.synchronize()
    # same images, same products: only the Gram of the two states may differ, in
    # the order of its FP64 sums
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy()) or torch.allclose(got, want, rtol=1e-6, atol=1e-6 * float(want.abs().max()))


def test_images_follow_a_rebind(S1000):
    """Steps on BF16, then on FP32 storage: equal to a fresh FP32 state from the
    iterate at the move."""
    c, k = ctx(), 20
    lo = sym.symnmf_S_load(c, to_dev(S1000, torch.float64), dtype=sym.S_BF16)
    hi = sym.symnmf_S_load(c, to_dev(S1000, torch.float64), dtype=sym.S_FP32)
    p = sym.symnmf_params_default(method=sym.MU, eps=2.0 ** -23)
    st = sym.symnmf_state_create(c, lo, k, p, to_dev(o.init_H(0.1, N, k, 3, as_float32=True)))
    for _ in range(2):
        sym.symnmf_step(c, lo, st, want_stats=False)
    H = sym.symnmf_state_read(c, st, 0, torch.empty(N, k, device=dev()))
    sym.symnmf_state_rebind(c, st, hi)
    fresh = sym.symnmf_state_create(c, hi, k, p, H)
    for _ in range(2):
        sym.symnmf_step(c, hi, st, want_stats=False)
        sym.symnmf_step(c, hi, fresh, want_stats=False)
    a = sym.symnmf_state_read(c, st, 0, torch.empty(N, k, device=dev()))
    b = sym.symnmf_state_read(c, fresh, 0, torch.empty(N, k, device=dev()))
    torch.cuda.synchronize()
    assert torch.allclose(a, b, rtol=1e-6, atol=1e-6 * float(b.abs().max()))
