"""Truncation with the output in the input's place, with and without room for all entries (one launch, and selection
and write apart): the same entries as in an array of its own."""
import ctypes as C

import numpy as np
import pytest

from paper_2312_01846_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n", [1, 900, 1025, 4000, 16384, 40001])
def test_in_place(n, noalloc):
    import torch

    from paper_2312_01846_amd import sfci

    h, g = synth.molecule_like(10, 20, 3)
    P = sfci.Problem(10, 5, 5, h, g)
    r, a = synth.random_sparse_vector(P.n_det, n, seed=n)
    M = (2 * n + 2) // 3
    wr, wa = (t.cpu().numpy() for t in P.topm(r.astype(np.int64), a, M))
    fn = getattr(sfci.load_library(), "sfci_topm_noalloc" if noalloc else "sfci_topm")
    for capacity in (n, M):
        vr = torch.as_tensor(r.astype(np.int64), device="cuda")
        va = torch.as_tensor(a, device="cuda")
        v = sfci._svec(vr, va)
        out = sfci.SVec(vr.data_ptr(), va.data_ptr(), 0, capacity)
        assert fn(P._h, C.byref(v), M, 0, 0, C.byref(out)) == 0
        assert out.nnz == wr.size
        assert np.array_equal(vr[:wr.size].cpu().numpy(), wr)
        assert np.array_equal(va[:wr.size].cpu().numpy(), wa)
