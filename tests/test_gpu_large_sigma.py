"""A truncated fast sigma of a space of 6.9e8 determinants leaves the N_det array out (dedup="auto"): the same
determinants as with it (dedup="dense"), amplitudes to rounding, the same counts, on both sides of the rule's limits."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2312_01846_amd import sfci

    h, g = synth.molecule_like(22, 44, 3)
    return sfci.Problem(22, 5, 5, h, g)


def _start(P, nnz, seed):
    r, a = synth.random_sparse_vector(P.n_det, nnz, seed=seed)
    return r.astype(np.int64), a


@pytest.mark.parametrize("nnz", [1, 300, 20000])
@pytest.mark.parametrize("kw", [dict(), dict(screen_eps=1e-4), dict(excite_eps=1e-5), dict(tie_band=True)])
def test_list_route_equals_dense(P, nnz, kw):
    r, a = _start(P, nnz, nnz)
    for M in (1, 1000, P.n_det // 1024, P.n_det // 1024 + 1):
        gr, ga, gs = P.sigma(r, a, M=M, **kw)
        dr, da, ds = P.sigma(r, a, M=M, dedup="dense", **kw)
        assert np.array_equal(gr.cpu().numpy(), dr.cpu().numpy())
        # sums of at most some thousand terms in another order
        assert np.allclose(ga.cpu().numpy(), da.cpu().numpy(), rtol=0, atol=1e-12 * np.abs(da.cpu().numpy()).max())
        assert gs["terms_emitted"] == ds["terms_emitted"] and gs["candidates"] == ds["candidates"]


def test_errors_as_before(P):
    from paper_2312_01846_amd import sfci

    r, a = _start(P, 50, 5)
    for bad in (np.array([5, 3]), np.array([1, 1]), np.array([0, P.n_det])):
        codes = []
        for d in ("auto", "dense"):
            with pytest.raises(sfci.SfciError) as e:
                P.sigma(bad.astype(np.int64), np.ones(2), M=100, dedup=d)
            codes.append(e.value.code)
        assert codes[0] == codes[1]
