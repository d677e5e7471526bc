"""The list iteration's sigma by target rows in fast mode: short rows in hash tables (one part, and many parts of
both table sizes), long rows through the tile kernel, against the iteration with the N_det array; unequal spins, no
doubles of one spin, screens, a truncation with exact ties."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

SPACES = [(8, 3, 3), (9, 1, 4), (9, 4, 1), (10, 5, 2), (12, 4, 4), (16, 2, 5)]


def _case(space, hubbard=False):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.hubbard_ring(n, 1.0, 4.0) if hubbard else synth.molecule_like(n, 2 * n, 3)
    P = sfci.Problem(n, na, nb, h, g)
    r, a = synth.random_sparse_vector(P.n_det, min(P.n_det // 2, 3000), seed=2)
    return P, r.astype(np.int64), a


# 0: every row through the tile kernel; the default; never the tile kernel
@pytest.mark.parametrize("heavy", ["0", None, "1000000000000"])
@pytest.mark.parametrize("space", SPACES)
def test_rows_match_dense_iteration(monkeypatch, space, heavy):
    if heavy is not None:
        monkeypatch.setenv("SFCI_LIST_HEAVY", heavy)
    P, r, a = _case(space)
    for kw in (dict(), dict(screen_eps=1e-4), dict(excite_eps=1e-5)):
        ref = P.lanczos(r, a, M=None, n_L=3, n_iter=3, want_T=True, **kw)
        out = P.lanczos(r, a, M=None, n_L=3, n_iter=3, want_T=True, no_dense=True, **kw)
        # a target sums some thousand terms in another order: 1e-12 of the largest element, ten times that after
        # two more applications
        assert np.allclose(out["T"], ref["T"], rtol=0, atol=1e-11 * np.abs(ref["T"]).max())
        assert np.allclose(out["S"], ref["S"], rtol=0, atol=1e-11)
        if not kw:
            assert out["stats"]["terms_emitted"] == ref["stats"]["terms_emitted"]


@pytest.mark.parametrize("heavy", ["0", "3000", "1000000000000"])
def test_truncation_with_exact_ties(monkeypatch, heavy):
    # one application to a determinant of the Hubbard ring: few distinct magnitudes, so the cut falls into a tie,
    # which the smaller ranks win whichever rows come first
    monkeypatch.setenv("SFCI_LIST_HEAVY", heavy)
    P, _, _ = _case((10, 5, 5), hubbard=True)
    for M in (3, 7, 11):
        ref = P.lanczos(np.array([0]), np.array([1.0]), M=M, n_L=3, n_iter=3, want_T=True)
        out = P.lanczos(np.array([0]), np.array([1.0]), M=M, n_L=3, n_iter=3, want_T=True, no_dense=True)
        assert np.array_equal(out["psi_rank"].cpu().numpy(), ref["psi_rank"].cpu().numpy())
        assert np.allclose(out["T"], ref["T"], rtol=0, atol=1e-12)
