"""Deterministic sigma without a sort (rows that fit in LDS): the same bits as the CPU oracle and as the sort path
(dedup="sort"), in spaces with no doubles, one alpha string, odd and unequal spins, a two-entry source, all entries,
zero elements, both screens, and rows longer than one group of beta singles."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

SPACES = [(5, 5, 2), (5, 2, 5), (6, 0, 3), (7, 3, 0), (9, 1, 4), (9, 4, 1), (8, 3, 3), (11, 5, 6), (17, 2, 5), (18, 5, 2),
          (12, 6, 6)]


def _problem(space, seed):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.hubbard_ring(n, 1.0, 4.0) if space == (12, 6, 6) else synth.molecule_like(n, 2 * n, seed)
    return sfci.Problem(n, na, nb, h, g), (n, na, nb, h, g)


def _same(x, y):
    assert np.array_equal(x[0].cpu().numpy(), y[0].cpu().numpy())
    assert np.array_equal(x[1].cpu().numpy(), y[1].cpu().numpy())


@pytest.mark.parametrize("space", SPACES)
@pytest.mark.parametrize("nnz", [2, 777, 20000])
def test_sigma_bits(orc, space, nnz):
    P, args = _problem(space, 7)
    r, a = synth.random_sparse_vector(P.n_det, min(nnz, P.n_det), seed=3)
    rt = r.astype(np.int64)
    got = P.sigma(rt, a, deterministic=True)
    ref = P.sigma(rt, a, deterministic=True, dedup="sort")
    _same(got, ref)
    assert got[2]["terms_emitted"] == ref[2]["terms_emitted"]
    wr, wa = orc.Problem(*args).sigma(r, a)
    assert np.array_equal(got[0].cpu().numpy().astype(np.uint64), wr)
    assert np.array_equal(got[1].cpu().numpy(), wa)
    for kw in (dict(screen_eps=1e-3), dict(excite_eps=1e-4), dict(M=max(1, wr.size // 3), screen_eps=1e-4)):
        x, y = (P.sigma(rt, a, deterministic=True, dedup=d, **kw) for d in ("auto", "sort"))
        _same(x, y)
        assert x[2]["terms_emitted"] == y[2]["terms_emitted"]
