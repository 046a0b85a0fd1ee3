"""The tail dependence build's rank, selection and angular kernels where they
change form: sample counts at the edges of the rank kernel's four sizes,
columns full of ties (including both zeros), equal radial norms at the
threshold, every sample kept, and column and row counts around the 64 x 64
tiles.  FP64 storage against the oracle."""
import numpy as np
import pytest

import oracle as o
import paper_2607_24518_amd as sym
import synth

pytestmark = pytest.mark.gpu

from gpu_util import ctx, stored_numpy, to_dev  # noqa: E402

# FP64 products of unit columns over at most 3277 rows, entries formed by one
# division and one root instead of a power: a few 2^-53 per entry
TOL = 1e-13


def _check(X, **kw):
    S = sym.symnmf_build_S(ctx(), to_dev(X), kind=sym.TPDM, dtype=sym.S_FP64, **kw)
    ref = o.tpdm(X, q=kw["q"], lower_tail=bool(kw["lower_tail"]), raw_marginals=bool(kw.get("raw_marginals", 0)))
    assert np.max(np.abs(stored_numpy(S) - ref)) <= TOL


@pytest.mark.parametrize("T", [2, 63, 65, 2048, 2049, 8192, 8193, 20480, 20481, 32768])
def test_ranks_at_the_kernel_sizes(T):
    X = np.random.default_rng(T).standard_t(3, size=(T, 3)).astype(np.float32)
    X[:, 1] = np.round(X[:, 1])                       # long runs of ties, -0.0 among them
    _check(X, q=1.0 if T < 100 else 0.1, lower_tail=1)
    _check(X, q=1.0 if T < 100 else 0.01, lower_tail=0)


@pytest.mark.parametrize("n,q", [(63, 0.05), (64, 0.064), (65, 0.065), (130, 0.2)])
def test_tiles_of_kept_rows_and_columns(n, q):
    _check(synth.tpdm_returns(2, T=1000, n=n, groups=4).X.numpy(), q=q, lower_tail=1)
    _check(synth.paper_benchmark(3, n, "tpdm", T=1000).X.numpy(), q=q, lower_tail=0, raw_marginals=1)


def test_equal_norms_keep_the_lower_samples():
    """Every sample appears four times, so the threshold falls inside a run of
    equal norms; the first copies are kept."""
    X = np.repeat(synth.paper_benchmark(5, 20, "tpdm", T=500).X.numpy(), 4, axis=0)
    X = X[np.random.default_rng(1).permutation(2000)]
    for q in (0.0125, 0.0505, 0.333):
        _check(X, q=q, lower_tail=0, raw_marginals=1)


def test_nonfinite_raw_panel_is_refused():
    X = synth.paper_benchmark(5, 20, "tpdm", T=500).X.numpy()
    for v in (np.nan, np.inf):
        X[400, 3] = v
        with pytest.raises(sym.SymnmfError) as e:
            sym.symnmf_build_S(ctx(), to_dev(X), kind=sym.TPDM, q=0.05, lower_tail=0, raw_marginals=1)
        assert e.value.code == sym.ENUMERIC
