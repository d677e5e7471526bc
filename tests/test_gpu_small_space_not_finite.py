"""A small space (H as a table) with an infinite integral: sigma of a vector that does not hold the orbital is finite
at every target, as the tile kernel gives it."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", [(8, 3, 3), (7, 3, 2)])
def test_infinite_integral(space):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.molecule_like(n, 2 * n, 3)
    h[n - 1, n - 1] = np.inf
    P = sfci.Problem(n, na, nb, h, g)
    r = np.arange(P.n_det, dtype=np.int64)
    A, B = (t.cpu().numpy() for t in P.unrank(r))
    r = r[((A | B) >> (n - 1)) & 1 == 0]
    a = np.random.default_rng(5).normal(size=r.size)
    for _ in range(2):
        gr, ga, gs = P.sigma(r, a)
        dr, da, ds = P.sigma(r, a, dedup="dense")
        assert np.isfinite(da.cpu().numpy()).all()
        assert np.array_equal(gr.cpu().numpy(), dr.cpu().numpy())
        # some hundred terms a sum, in another order
        assert np.allclose(ga.cpu().numpy(), da.cpu().numpy(), rtol=0, atol=1e-12 * np.abs(da.cpu().numpy()).max())
        assert gs["terms_emitted"] == ds["terms_emitted"]
