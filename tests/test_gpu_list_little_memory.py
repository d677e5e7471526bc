"""A truncated sigma without an N_det array on a device with 3 GiB free, of a vector in the last alpha rows: a bound
from the first rows lets nearly every entry of the others join the candidates, more than fit at once.  The same
determinants as with all of the memory, by lists and by the N_det array."""
import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["last", "first"])
def test_candidates_in_parts(where):
    import torch

    from paper_2312_01846_amd import sfci

    n, k, M = 22, 5, 200000
    h, g = synth.molecule_like(n, 2 * n, 3)
    n_beta = 26334
    rng = np.random.default_rng(4)
    ra, rb = (np.floor(rng.exponential(2000.0, 400000)).astype(np.int64) % n_beta for _ in range(2))
    r = np.unique(ra * n_beta + rb)
    if where == "last":
        r = np.sort(n_beta * n_beta - 1 - r)
    a = rng.normal(size=r.size)
    got = []
    for little, dedup in ((False, "dense"), (False, "auto"), (True, "auto")):
        P = sfci.Problem(n, k, k, h, g)
        P.sigma(r[:1000], a[:1000], M=1000)  # tables
        torch.cuda.empty_cache()
        free, _ = torch.cuda.mem_get_info()
        hog = torch.empty(max(1, free - (3 << 30)) if little else 1, dtype=torch.uint8, device="cuda")
        try:
            R, A, S = P.sigma(r, a, M=M, dedup=dedup)
            got.append((R.cpu().numpy(), A.cpu().numpy(), S["candidates"], S["terms_emitted"]))
        finally:
            del hog
            P.close()
            torch.cuda.empty_cache()
    for x in got[1:]:
        assert np.array_equal(x[0], got[0][0]) and x[2:] == got[0][2:]
        # sums of at most some thousand terms in another order
        assert np.allclose(x[1], got[0][1], rtol=0, atol=1e-12 * np.abs(got[0][1]).max())
