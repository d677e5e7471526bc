"""Deterministic sigma without a sort where a string has 64 beta singles or more (a second group of lanes, with the
beta-unchanged target added by itself): the same bits as the CPU oracle and as the sort path, also with an amplitude
that is not finite."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

# n_beta (n - n_beta) = 63, 64, 66, 66 (rows of 12 376 slots), 65, 75, 68, 66
SPACES = [(16, 2, 7), (20, 3, 4), (17, 2, 6), (17, 2, 11), (18, 3, 5), (20, 2, 5), (21, 3, 4), (25, 4, 3)]


@pytest.fixture(scope="module", params=SPACES, ids=str)
def case(request, orc):
    from paper_2312_01846_amd import sfci

    n, na, nb = request.param
    h, g = synth.molecule_like(n, 2 * n, 7)
    return sfci.Problem(n, na, nb, h, g), orc.Problem(n, na, nb, h, g)


def _vector(P, nnz, seed):
    """Entries in a few long source rows and all over the space."""
    rng = np.random.default_rng(seed)
    r = np.concatenate([rng.integers(0, min(P.n_det, 20 * nnz), nnz // 2), rng.integers(0, P.n_det, nnz - nnz // 2)])
    r = np.unique(r).astype(np.uint64)
    return r, rng.normal(size=r.size)


def _same(got, ref):
    assert np.array_equal(got[0].cpu().numpy(), ref[0].cpu().numpy())
    assert np.array_equal(got[1].cpu().numpy(), ref[1].cpu().numpy(), equal_nan=True)
    assert got[2]["terms_emitted"] == ref[2]["terms_emitted"]


@pytest.mark.parametrize("nnz", [2, 300, 4000])
def test_bits(case, nnz):
    P, Po = case
    r, a = _vector(P, nnz, nnz)
    got = P.sigma(r.astype(np.int64), a, deterministic=True)
    _same(got, P.sigma(r.astype(np.int64), a, deterministic=True, dedup="sort"))
    wr, wa = Po.sigma(r, a)
    assert np.array_equal(got[0].cpu().numpy().astype(np.uint64), wr)
    assert np.array_equal(got[1].cpu().numpy(), wa)
    kw = dict(excite_eps=1e-3, screen_eps=1e-3)
    _same(*(P.sigma(r.astype(np.int64), a, deterministic=True, dedup=d, **kw) for d in ("auto", "sort")))


def test_bits_not_finite(case):
    P, _ = case
    r, a = _vector(P, 300, 5)
    a[r.size // 3] = np.inf
    a[r.size // 2] = 0.0
    for kw in (dict(), dict(excite_eps=1e-3)):
        _same(*(P.sigma(r.astype(np.int64), a, deterministic=True, dedup=d, **kw) for d in ("auto", "sort")))
