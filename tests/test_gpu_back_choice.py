"""The backward of sigma where the entries decide between rows and the walk per source: vectors gathered in few alpha
rows and spread-out ones, with cotangents in few and many rows, against the CPU oracle."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

SPACES = [(12, 4, 4), (18, 9, 1), (16, 2, 4), (9, 0, 4), (24, 1, 3)]


def _vector(n_det, n_beta, nnz, rows, seed):
    rng = np.random.default_rng(seed)
    n_alpha = n_det // n_beta
    r = np.unique(rng.integers(0, min(rows, n_alpha), 4 * nnz) * n_beta + rng.integers(0, n_beta, 4 * nnz))
    r = np.sort(rng.permutation(r)[:nnz]).astype(np.uint64)
    return r, rng.normal(size=r.size)


@pytest.mark.parametrize("space", SPACES, ids=str)
@pytest.mark.parametrize("rows", [40, 1 << 30])
@pytest.mark.parametrize("s_rows", [10, 1 << 30])
def test_matches_oracle(orc, space, rows, s_rows):
    import math

    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.molecule_like(n, 2 * n, 7)
    P, n_beta = sfci.Problem(n, na, nb, h, g), math.comb(n, nb)
    vr, va = _vector(P.n_det, n_beta, 5000, rows, 5)
    sr, sa = _vector(P.n_det, n_beta, 3000, s_rows, 6)
    got = P.sigma_backward(vr.astype(np.int64), va, sr.astype(np.int64), sa)
    want = orc.Problem(n, na, nb, h, g).backward(vr, va, sr, sa)
    # the tolerances of the general backward's parity test
    assert np.allclose(got[0].cpu().numpy(), want[0], rtol=1e-12, atol=1e-12)
    assert np.allclose(got[1].cpu().numpy(), want[1], rtol=1e-9, atol=1e-11)
    assert np.allclose(got[2].cpu().numpy(), want[2], rtol=1e-9, atol=1e-11)
