"""The list iteration's sigma with few terms, on both sides of the line between the sort path and the rows (few
alpha strings and many, just below and above the limit of terms): the sort path runs, and only there, and T, S and
Psi are those of the iteration with the N_det array."""
import math

import numpy as np
import pytest
import torch

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


def _terms(n, na, nb):
    one = lambda k: (k * (n - k), math.comb(k, 2) * math.comb(n - k, 2))
    (sa, da), (sb, db) = one(na), one(nb)
    return 1 + sa + sb + da + db + sa * sb


# 4 845 and 8 568 alpha strings; terms per sigma below and above 8e6
@pytest.mark.parametrize("space,terms", [((12, 6, 6), 1.8e6), ((20, 4, 4), 7.0e6), ((20, 4, 4), 9.0e6),
                                         ((18, 5, 5), 1.0e6), ((16, 2, 5), 1e5), ((20, 1, 6), 9e4)], ids=str)
def test_matches_dense_iteration(monkeypatch, space, terms):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.molecule_like(n, 2 * n, 3)
    P = sfci.Problem(n, na, nb, h, g)
    r, a = synth.random_sparse_vector(P.n_det, max(1, int(terms / _terms(n, na, nb))), seed=2)
    run = lambda **kw: P.lanczos(r.astype(np.int64), a, M=None, n_L=1, n_iter=1, want_T=True, **kw)
    ref, out = run(), run(no_dense=True)
    # a target sums some thousand terms in another order: 1e-12 of the largest element
    assert np.allclose(out["T"], ref["T"], rtol=0, atol=1e-12 * np.abs(ref["T"]).max())
    assert out["stats"]["terms_emitted"] == ref["stats"]["terms_emitted"]
    # the sort path takes its tuple buffers in its first two runs, so asking for it afterwards takes memory or not
    run(no_dense=True)
    by_sort = terms < 8e6 and math.comb(n, na) <= 8192
    free = torch.cuda.mem_get_info()[0]
    monkeypatch.setenv("SFCI_LIST_SIGMA", "sort")
    run(no_dense=True)
    assert (torch.cuda.mem_get_info()[0] == free) == by_sort
