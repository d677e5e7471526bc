"""The correction taken from the dense accumulator, row by row: unequal spins, rows of one entry, row lengths
around the workgroup's 256 and 1 024, a spin with no electrons.  E0 and the external determinants against the
deterministic list form; E2 against the formula at the E0 that came with it (a random vector's E0 lies among
the diagonal elements, so E2 amplifies E0's last bits), with H Psi from the deterministic sigma and H_kk
added in the diagonal element's order."""
import math

import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


def _occupied(bits, n, k):
    out = np.zeros((bits.size, k), dtype=np.int64)
    at = np.zeros(bits.size, dtype=np.int64)
    for p in range(n):
        on = np.nonzero((bits >> p) & 1)[0]
        out[on, at[on]] = p
        at[on] += 1
    return out


def _diagonal(h, g, A, B):
    e = np.zeros(A.shape[0])
    for S in (A, B):
        for t in range(S.shape[1]):
            e = e + h[S[:, t], S[:, t]]
    for S in (A, B):
        for t in range(S.shape[1]):
            for u in range(t + 1, S.shape[1]):
                p, q = S[:, t], S[:, u]
                e = e + (g[p, p, q, q] - g[p, q, q, p])
    for t in range(A.shape[1]):
        for u in range(B.shape[1]):
            e = e + g[A[:, t], A[:, t], B[:, u], B[:, u]]
    return e


@pytest.mark.parametrize("n,na,nb,nnz", [(8, 3, 3, 1), (12, 3, 2, 40), (13, 2, 5, 500), (14, 5, 3, 3000),
                                         (10, 0, 3, 30), (10, 3, 0, 30), (9, 9, 4, 20), (16, 2, 4, 7000)])
def test_dense_form(n, na, nb, nnz):
    from paper_2312_01846_amd import sfci

    h, g = synth.molecule_like(n, 2 * n, 11)
    P = sfci.Problem(n, na, nb, h, g)
    r, a = synth.random_sparse_vector(P.n_det, nnz, seed=nnz)
    r = r.astype(np.int64)
    e0, e2, ne = P.pt2(r, a)
    d0, _, de = P.pt2(r, a, deterministic=True)
    assert ne == de
    assert abs(e0 - d0) <= 1e-11 * max(1.0, abs(d0))
    tr, ta, _ = P.sigma(r, a, M=None, deterministic=True)
    ab, bb = P.unrank(tr)
    tr, ta = tr.cpu().numpy(), ta.cpu().numpy()
    ext = ~np.isin(tr, r)
    hkk = _diagonal(h, g, _occupied(ab.cpu().numpy(), n, na), _occupied(bb.cpu().numpy(), n, nb))
    terms = ta[ext] ** 2 / (e0 - hkk[ext])
    want = math.fsum(terms) / math.fsum(a * a)
    # each y is good to ~1e-14 of itself or of the largest, each term to twice that
    assert abs(e2 - want) <= 1e-10 * max(1.0, abs(want))
    # the accumulator is clear again
    sr, sa, _ = P.sigma(r, a, M=None)
    assert np.array_equal(sr.cpu().numpy(), tr)
    assert np.allclose(sa.cpu().numpy(), ta, rtol=1e-10, atol=1e-12)
