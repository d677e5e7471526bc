"""The row form of the backward (vbar with both integral gradients) against the CPU oracle: rows of one entry
and of many 64-entry chunks, more than 64 beta singles, several tiles per row, a spin with one electron or none
or no virtuals, a cotangent that misses rows."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

# (n, n_alpha, n_beta, nnz(v), nnz(sbar), rows of sbar kept)
CASES = {"one": (9, 2, 3, 1, 1500, 1.0), "long rows": (11, 1, 5, 3000, 2500, 1.0),
         "wide beta": (18, 1, 5, 400, 30000, 1.0), "tiles": (14, 2, 5, 1500, 20000, 1.0),
         "beta none": (12, 4, 0, 200, 300, 1.0), "alpha none": (12, 0, 4, 200, 300, 1.0),
         "alpha full": (7, 7, 3, 30, 30, 1.0), "beta one": (13, 4, 1, 900, 4000, 1.0),
         "sparse rows": (12, 4, 4, 2000, 20000, 0.3)}


@pytest.mark.parametrize("form", ["1", "0"])
@pytest.mark.parametrize("name", list(CASES))
def test_backward_rows_match_oracle(name, form, monkeypatch):
    import oracle

    from paper_2312_01846_amd import sfci

    monkeypatch.setenv("SFCI_BACK_ROWS", form)  # the rows, and the walk per source that short inputs take
    n, na, nb, nv, ns, rows = CASES[name]
    if name == "tiles":
        monkeypatch.setenv("SFCI_TILE_MAX", "1024")
    h, g = synth.molecule_like(n, 2 * n, 7)
    P = sfci.Problem(n, na, nb, h, g)
    Po = oracle.Problem(n, na, nb, h, g)
    vr, va = synth.random_sparse_vector(P.n_det, nv, 5)
    sr, sa = synth.random_sparse_vector(P.n_det, ns, 6)
    if rows < 1.0:
        n_beta_strings = P.n_det // Po_rows(n, na)
        keep = np.random.default_rng(8).random(Po_rows(n, na)) < rows
        on = keep[(sr // np.uint64(n_beta_strings)).astype(np.int64)]
        sr, sa = sr[on], sa[on]
    vbar, dh, dg = P.sigma_backward(vr.astype(np.int64), va, sr.astype(np.int64), sa)
    ov, oh, og = Po.backward(vr, va, sr, sa)
    # the tolerances of the general backward's parity test
    assert np.allclose(vbar.cpu().numpy(), ov, rtol=1e-12, atol=1e-12)
    assert np.allclose(dh.cpu().numpy(), oh, rtol=1e-9, atol=1e-11)
    assert np.allclose(dg.cpu().numpy(), og, rtol=1e-9, atol=1e-11)


def Po_rows(n, na):
    import math

    return math.comb(n, na)
