"""The S-building products at the edges of their tile order (tile rows from 2 to
18, ragged last blocks of 8 x 8 tiles), for row panels that start at any column,
and into memory that held something else: every entry of the storage, padding
included, and every padding entry of the scratch has to be written.

Oracle: FP64 correlations.  FP32 storage: T products of unit columns, random
walk, 4 sqrt(T) 2^-24; BF16 and FP8 add their rounding (2^-8 and 2^-4 of the
largest entry of a scale panel's rows, at most 1)."""
import numpy as np
import pytest
import torch

import paper_2607_24518_amd as sym

pytestmark = pytest.mark.gpu

from gpu_util import ctx, dev, from_dev, stored_numpy, untile  # noqa: E402

E = {"fp32": 4, "bf16": 8, "fp8": 16}
TYPE = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn, "fp64": torch.float64}


def _dirty(nbytes, device):
    return torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=device)


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8", "fp64"])
@pytest.mark.parametrize("n,row0,rows,T", [(3, 0, 3, 5), (256, 0, 256, 16), (300, 0, 300, 33), (700, 0, 700, 17),
                                           (1100, 0, 1100, 40), (2300, 0, 2300, 31), (900, 1, 600, 20),
                                           (700, 513, 187, 47)])
def test_correlations(dtype, n, row0, rows, T, monkeypatch):
    g = torch.Generator("cuda").manual_seed(n + T)
    X = torch.randn(T, n, generator=g, device=dev()) + 0.5 * torch.randn(T, 1, generator=g, device=dev())
    c = sym.symnmf_create(0)
    monkeypatch.setattr(sym, "_alloc_bytes", _dirty)
    kw = dict(kind=sym.ABS_CORR, dtype=sym.DTYPES[dtype], row0=row0, rows=rows)
    work = _dirty(sym.symnmf_build_S_workspace(n, T, **kw) + 4096, dev())
    sym.symnmf_set_workspace(c, work)
    S = sym.symnmf_build_S(c, X, **kw)
    sym.symnmf_set_workspace(c)
    sym.symnmf_destroy(c)
    x = from_dev(X).astype(np.float64)
    z = x - x.mean(0)
    z /= np.sqrt((z * z).sum(0))
    ref = np.abs(z[:, row0:row0 + rows].T @ z)
    ref[np.arange(rows), row0 + np.arange(rows)] = 1.0
    got = stored_numpy(S)
    tol = {"fp64": 1e-12, "fp32": 0.0, "bf16": 2.0 ** -8, "fp8": 2.0 ** -4}[dtype]
    assert np.max(np.abs(got - ref)) <= tol + (0 if dtype == "fp64" else 4 * np.sqrt(T) * 2.0 ** -24)
    if rows == n and dtype != "fp8":
        assert np.array_equal(got, got.T)
    d = S.desc
    item = torch.empty(0, dtype=TYPE[dtype]).element_size()
    flat = S.buf[: d.rows_pad * d.ld * item].view(TYPE[dtype])
    full = flat.view(d.rows_pad, d.ld) if dtype == "fp64" else untile(flat, d.rows_pad, d.ld, E[dtype])
    full = full.double()
    assert torch.all(full[rows:] == 0) and torch.all(full[:, n:] == 0)
    assert abs(d.fro2_stored - float((got * got).sum())) <= 1e-9 * d.fro2_stored
