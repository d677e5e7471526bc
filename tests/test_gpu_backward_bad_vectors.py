"""The backward of sigma leaves its outputs alone when a vector is bad (a rank out of range, ranks not ascending),
whichever of the two it is and on each of its routes, and works afterwards."""
import ctypes as C

import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", ["rows", "sources", "tiles"])
def test_outputs_untouched(monkeypatch, route):
    import torch

    from paper_2312_01846_amd import sfci

    monkeypatch.setenv("SFCI_BACK_ROWS", "1" if route == "rows" else "0")
    n = 8
    h, g = synth.molecule_like(n, 2 * n, 3)
    P = sfci.Problem(n, 3, 3, h, g)
    r, a = synth.random_sparse_vector(P.n_det, 300, seed=2)
    s, b = synth.random_sparse_vector(P.n_det, 200, seed=3)
    dev = lambda x, t: torch.as_tensor(np.asarray(x).astype(t), device="cuda")
    vr, va, sr, sa = dev(r, np.int64), dev(a, np.float64), dev(s, np.int64), dev(b, np.float64)
    out = [torch.full((m,), 7.0, dtype=torch.float64, device="cuda") for m in (r.size, n**2, n**4)]

    def call(v_rank, s_rank):
        ptr = [x.data_ptr() for x in out]
        if route == "tiles":
            ptr[0] = None
        return sfci.load_library().sfci_sigma_backward(P._h, C.byref(sfci._svec(v_rank, va)),
                                                       C.byref(sfci._svec(s_rank, sa)), *ptr)

    for good, which in ((vr, 0), (sr, 1)):
        for bad_rank, code in ((P.n_det, -2), (int(good[-2]), -3)):
            x = good.clone()
            x[-1] = bad_rank
            assert call(*((x, sr) if which == 0 else (vr, x))) == code
            torch.cuda.synchronize()
            assert all(bool((t == 7.0).all()) for t in out)
    assert call(vr, sr) == 0
    vb, dh, dg = P.sigma_backward(vr, va, sr, sa)
    got = [t.cpu().numpy() for t in out]
    for x, y in zip(got[1:] if route == "tiles" else got, (dh, dg) if route == "tiles" else (vb, dh, dg)):
        y = y.cpu().numpy().ravel()
        # at most some thousand terms a sum, in another order
        assert np.all(np.abs(x - y) <= 1e-11 * np.abs(y).max())
