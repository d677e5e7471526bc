"""The backward of sigma with v_bar in the place of v's amplitudes: the same sums as with an array of its own."""
import ctypes as C

import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", ["1", "0"])
def test_vbar_over_amplitudes(orc, monkeypatch, rows):
    import torch

    from paper_2312_01846_amd import sfci

    monkeypatch.setenv("SFCI_BACK_ROWS", rows)
    n = 10
    h, g = synth.molecule_like(n, 2 * n, 3)
    P = sfci.Problem(n, 4, 3, h, g)
    r, a = synth.random_sparse_vector(P.n_det, 5000, seed=2)
    s, b = synth.random_sparse_vector(P.n_det, 4000, seed=3)
    vr, sr = (torch.as_tensor(x.astype(np.int64), device="cuda") for x in (r, s))
    va, sa = (torch.as_tensor(x, device="cuda") for x in (a, b))
    dh = torch.empty(n**2, dtype=torch.float64, device="cuda")
    dg = torch.empty(n**4, dtype=torch.float64, device="cuda")
    v = sfci._svec(vr, va)
    assert sfci.load_library().sfci_sigma_backward(P._h, C.byref(v), C.byref(sfci._svec(sr, sa)), va.data_ptr(),
                                                   dh.data_ptr(), dg.data_ptr()) == 0
    wv, wh, wg = orc.Problem(n, 4, 3, h, g).backward(r, a, s, b)
    # the tolerances of the general backward's parity test
    assert np.allclose(va.cpu().numpy(), wv, rtol=1e-12, atol=1e-12)
    assert np.allclose(dh.cpu().numpy(), wh.ravel(), rtol=1e-9, atol=1e-11)
    assert np.allclose(dg.cpu().numpy(), wg.ravel(), rtol=1e-9, atol=1e-11)
