"""Deterministic sigma of a space of 6.0e8 determinants, truncated to a small part of it: the bits of the sort path,
on both sides of the in-order rule's limit (a quarter as many terms as determinants: 16 928 entries)."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2312_01846_amd import sfci

    h, g = synth.molecule_like(20, 40, 3)
    return sfci.Problem(20, 6, 5, h, g)


@pytest.mark.parametrize("nnz", [10000, 20000])
@pytest.mark.parametrize("kw", [dict(), dict(tie_band=True), dict(screen_eps=1e-4)])
def test_bits_of_the_sort_path(P, nnz, kw):
    r, a = synth.random_sparse_vector(P.n_det, nnz, seed=nnz)
    r = r.astype(np.int64)
    for M in (1000, 100000):
        x, y = (P.sigma(r, a, M=M, deterministic=True, dedup=d, **kw) for d in ("auto", "sort"))
        assert np.array_equal(x[0].cpu().numpy(), y[0].cpu().numpy())
        assert np.array_equal(x[1].cpu().numpy(), y[1].cpu().numpy())
        assert x[2]["terms_emitted"] == y[2]["terms_emitted"] and x[2]["candidates"] == y[2]["candidates"]
