"""The tile kernel with eight wavefronts, two workgroups to a compute unit: a single vector of at most one entry per
alpha row (its limit and one more entry), spaces at the limits of the rule (256 orbital pairs and more, rows too long
for two), both screens; several instances in one launch."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu

# C(12,4) = 495, C(16,5) = 4 368, 23 and 24 virtuals (253 and 276 pairs), beta rows of 5 985 (too long for two)
SPACES = [(12, 4, 4), (16, 5, 2), (25, 2, 3), (26, 2, 2), (21, 2, 4), (9, 4, 1), (7, 3, 0)]


def _problem(space):
    from paper_2312_01846_amd import sfci

    n, na, nb = space
    h, g = synth.molecule_like(n, 2 * n, 4)
    return sfci.Problem(n, na, nb, h, g), (n, na, nb, h, g)


@pytest.mark.parametrize("space", SPACES)
def test_sigma_matches_oracle(orc, space):
    P, args = _problem(space)
    Po = orc.Problem(*args)
    from math import comb

    for nnz in (1, comb(space[0], space[1]), comb(space[0], space[1]) + 1):
        r, a = synth.random_sparse_vector(P.n_det, min(nnz, P.n_det // 2), seed=nnz)
        for eps in (0.0, 1e-3):
            wr, wa = Po.sigma(r, a) if eps == 0.0 else (None, None)
            gr, ga, st = P.sigma(r.astype(np.int64), a, dedup="dense", screen_eps=eps)
            sr, sa, ss = P.sigma(r.astype(np.int64), a, dedup="sort", screen_eps=eps)
            # sums of at most some thousand terms below max|H| |a| in another order
            assert np.array_equal(gr.cpu().numpy(), sr.cpu().numpy())
            assert np.allclose(ga.cpu().numpy(), sa.cpu().numpy(), rtol=0, atol=1e-11 * np.abs(sa.cpu().numpy()).max())
            assert st["terms_emitted"] == ss["terms_emitted"]
            if eps == 0.0:
                assert np.array_equal(gr.cpu().numpy().astype(np.uint64), wr)
                assert np.all(np.abs(ga.cpu().numpy() - wa) <= 1e-11 * np.abs(wa).max())


def test_instances_match_single_iterations():
    from paper_2312_01846_amd import sfci

    n, na, nb = 14, 4, 4
    probs = [sfci.Problem(n, na, nb, *synth.molecule_like(n, 2 * n, s)) for s in (1, 2, 3)]
    start = (np.array([0], dtype=np.int64), np.array([1.0]))
    Ms = [700, 5000, 40000]
    out = sfci.Batch(probs).lanczos([start] * 3, Ms, n_L=5, n_iter=5, want_grad=False, tie_band=True)
    for p, M, e in zip(probs, Ms, out["energies"]):
        ref = p.lanczos(*start, M=M, n_L=5, n_iter=5, tie_band=True)
        assert np.allclose(e, ref["energies"], rtol=0, atol=1e-9)
