"""The list iteration's sigma of vectors that gather in a few alpha strings of spaces with long beta rows, where the
sort path is the faster one, and of spread-out ones, around the line between few and many alpha strings: T is that of
the iteration with the N_det array."""
import math

import numpy as np
import pytest
import torch

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


# by_sort: long rows in hash tables (an alpha single of two of the six strings: 43 000 terms, six parts)
@pytest.mark.parametrize("space,rows,nnz,by_sort", [((24, 2, 8), 6, 1000, True), ((24, 2, 8), 1 << 30, 3000, False),
                                                    ((20, 3, 10), 2, 2000, False), ((16, 7, 7), 1 << 30, 2000, False),
                                                    ((16, 7, 7), 2, 1500, False)], ids=str)
def test_matches_dense_iteration(monkeypatch, space, rows, nnz, by_sort):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.molecule_like(n, 2 * n, 3)
    P, n_beta = sfci.Problem(n, na, nb, h, g), math.comb(n, nb)
    rng = np.random.default_rng(5)
    at = rng.integers(0, min(rows, math.comb(n, na)), 2 * nnz) * n_beta + rng.integers(0, n_beta, 2 * nnz)
    r = np.sort(rng.permutation(np.unique(at))[:nnz]).astype(np.int64)
    a = rng.normal(size=r.size)
    run = lambda **kw: P.lanczos(r, a, M=None, n_L=1, n_iter=1, want_T=True, **kw)
    ref, out = run(), run(no_dense=True)
    # a target sums some thousand terms in another order: 1e-12 of the largest element
    assert np.allclose(out["T"], ref["T"], rtol=0, atol=1e-12 * np.abs(ref["T"]).max())
    assert out["stats"]["terms_emitted"] == ref["stats"]["terms_emitted"]
    if by_sort:
        # the sort path takes its tuple buffers in its first two runs, so asking for it afterwards takes none
        run(no_dense=True)
        free = torch.cuda.mem_get_info()[0]
        monkeypatch.setenv("SFCI_LIST_SIGMA", "sort")
        run(no_dense=True)
        assert torch.cuda.mem_get_info()[0] == free
