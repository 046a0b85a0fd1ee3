"""f(H) of a float32 H at ranks other than 16 and 32: every product and sum in
FP64, so the value is that of the same H handed over in float64, up to the
order of FP64 sums; every storage type, each number of 16-column blocks, one
and several units per work-group, row panels.

Tolerance: f = ||S||^2 - 2 tr(H^T S H) + ||H^T H||^2, each entry of S H and of
H^T H a sum of n terms and the traces sums of those, all of one sign here: FP64
sums in any order differ by at most about n eps of the terms' size."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev  # noqa: E402


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,row0,rows,k", [(37, 0, 37, 1), (256, 0, 256, 15), (257, 0, 257, 17), (700, 0, 700, 64),
                                           (1500, 300, 513, 33), (2100, 0, 2100, 49), (6100, 0, 6100, 8),
                                           (7000, 0, 7000, 48), (6200, 0, 6200, 64)])
def test_equals_the_float64_form(dtype, n, row0, rows, k):
    c = ctx()
    g = torch.Generator("cuda").manual_seed(n + k)
    X = torch.randn(60, n, generator=g, device=dev()) + torch.randn(60, 1, generator=g, device=dev())
    S = sym.symnmf_build_S(c, X, dtype=sym.DTYPES[dtype], row0=row0, rows=rows, fp8_panel_rows=128)
    H = torch.rand(n, k, generator=g, device=dev()) * (torch.rand(n, k, generator=g, device=dev()) < 0.5) * 0.2
    f32, E32 = sym.symnmf_objective(c, S, H, k)
    f64, E64 = sym.symnmf_objective(c, S, H.double(), k)
    Hd = H.double()
    gram, own = Hd.T @ Hd, Hd[row0:row0 + rows].T @ Hd[row0:row0 + rows]
    fro2, hh = S.desc.fro2_stored, float((own * gram).sum())
    # |tr(H_own^T S H)| = |<S, H_own H^T>| <= ||S|| ||H_own H^T||
    tol = n * 2.0 ** -52 * (fro2 + 2.0 * np.sqrt(fro2 * hh) + hh)
    print(f"{dtype} n={n} rows={rows} k={k}: difference {abs(f32 - f64) / fro2:.2e} of ||S||^2, bound {tol / fro2:.2e}")
    assert abs(f32 - f64) <= tol
    assert abs(E32 - E64) <= tol / fro2
