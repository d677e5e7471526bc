"""A sigma that fails for want of device memory once its sums stand in the N_det array leaves the problem usable: the
next sigma gives what it gave before."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


def test_sigma_after_no_memory():
    import torch

    from paper_2312_01846_amd import sfci

    # 6.9e8 determinants: an array of 5.5 GB, and up to 2 x 6.9 GB of candidates when nearly all are kept
    n, k = 22, 5
    h, g = synth.molecule_like(n, 2 * n, 3)
    P = sfci.Problem(n, k, k, h, g)
    r, a = (x for x in synth.random_sparse_vector(P.n_det, 10, seed=1))
    R, A = (x for x in synth.random_sparse_vector(P.n_det, 300000, seed=2))
    small = lambda: [t.cpu().numpy() for t in P.sigma(r.astype(np.int64), a, M=1000, dedup="dense")[:2]]
    want = small()
    P.sigma(R.astype(np.int64), A, M=1000, dedup="dense")  # every other workspace at its size
    free, _ = torch.cuda.mem_get_info()
    hog = torch.empty(free - (4 << 30), dtype=torch.uint8, device="cuda")
    try:
        with pytest.raises(sfci.SfciError) as e:
            P.sigma(R.astype(np.int64), A, M=P.n_det - 1, dedup="dense", capacity=16)
        assert e.value.code == -5
    finally:
        del hog
        torch.cuda.empty_cache()
    got = small()
    assert np.array_equal(got[0], want[0])
    # sums of a few terms, in another order
    assert np.allclose(got[1], want[1], rtol=0, atol=1e-13 * np.abs(want[1]).max())
