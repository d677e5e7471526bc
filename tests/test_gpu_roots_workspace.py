"""Deterministic iteration with a projected root whose H Psi comes from the in-order kernel while the truncated basis
vectors go through the sort path: H Psi is a longer list than any sigma of the iteration, in the same workspace.  The
oracle's bits."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


def test_root_longer_than_the_basis(orc):
    from paper_2312_01846_amd import sfci

    # 7.5e7 determinants, 6 710 terms a source: from 2 800 entries on in order, below by the sort path
    n, na, nb, M = 20, 4, 5, 300
    h, g = synth.molecule_like(n, 2 * n, 11)
    P, Po = sfci.Problem(n, na, nb, h, g), orc.Problem(n, na, nb, h, g)
    rr, ra = synth.random_sparse_vector(P.n_det, 3000, seed=4)
    r0, a0 = synth.random_sparse_vector(P.n_det, 40, seed=5)
    ref = Po.lanczos(r0.astype(np.uint64), a0, M, 3, 3, roots=[(rr.astype(np.uint64), ra)])
    out = P.lanczos(r0.astype(np.int64), a0, M=M, n_L=3, n_iter=3, deterministic=True,
                    roots=[(rr.astype(np.int64), ra)])
    assert np.array_equal(out["energies"], ref["energies"])
    assert np.array_equal(out["psi_rank"].cpu().numpy().astype(np.uint64), ref["psi_rank"])
    assert np.array_equal(out["psi_amp"].cpu().numpy(), ref["psi_amp"])
