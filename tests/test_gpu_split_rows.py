"""The tile kernel's alpha-single source rows of more than 256 entries, listed as several records: rows of 256, 257 and
every beta string, one tile and several tiles per row (with and without the alpha-beta item lists), against the sort
path; zero elements and the excitation screen."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", ["one", "several", "several, no lists"])
@pytest.mark.parametrize("space,hubbard", [((14, 2, 5), False), ((14, 5, 5), False), ((12, 6, 6), True)])
def test_long_rows(monkeypatch, space, hubbard, tiles):
    from math import comb

    from paper_2312_01846_amd import sfci

    if tiles != "one":
        monkeypatch.setenv("SFCI_TILE_MAX", "1024")
    if tiles == "several, no lists":
        monkeypatch.setenv("SFCI_AB_LISTS", "0")
    n, na, nb = space
    h, g = synth.hubbard_ring(n, 1.0, 4.0) if hubbard else synth.molecule_like(n, 2 * n, 8)
    P = sfci.Problem(n, na, nb, h, g)
    Nb = comb(n, nb)
    rng = np.random.default_rng(1)
    rows = []
    for k in range(comb(n, na)):  # row lengths 255 ... 257, 511 ... 513, all, some and none in turn
        ln = [255, 256, 257, 511, 512, 513, Nb, 3, 0][k % 9]
        rows.append(k * Nb + np.sort(rng.choice(Nb, min(ln, Nb), replace=False)))
    r = np.concatenate(rows).astype(np.int64)
    a = rng.standard_normal(r.size) / np.sqrt(r.size)
    for kw in (dict(), dict(excite_eps=1e-5)):
        gr, ga, gs = P.sigma(r, a, dedup="dense", **kw)
        sr, sa, ss = P.sigma(r, a, dedup="sort", **kw)
        gr, ga, sr, sa = (x.cpu().numpy() for x in (gr, ga, sr, sa))
        assert gs["terms_emitted"] == ss["terms_emitted"]
        # some thousand terms per target in another order; an exact zero of one order may be a rounding rest of the other
        G, S = np.zeros(P.n_det), np.zeros(P.n_det)
        G[gr], S[sr] = ga, sa
        assert np.allclose(G, S, rtol=0, atol=1e-11 * np.abs(S).max())
