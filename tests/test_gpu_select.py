"""Truncation against a plain sort, at the sizes where the selection changes its path: one workgroup up to
16 384 entries, segments of 1 024 up to 4 Mi entries, of 4 096 beyond; and where many entries share the
leading bits of the M-th one (its bin holds more than 2 048)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BAND = 1.0 - 2.0 ** -36
SLACK = 256


@pytest.fixture(scope="module")
def P():
    from paper_2312_01846_amd import sfci

    return sfci.Problem(20, 4, 4, np.zeros((20, 20)), np.zeros(20 ** 4))


def _expected(r, a, M, band):
    nz = np.nonzero(a)[0]
    if M >= nz.size:
        return r[nz], a[nz]
    by = nz[np.argsort(-np.abs(a[nz]), kind="stable")]  # ranks ascend, so ties stay in rank order
    k = M
    if band and M > 0:
        more = int(np.count_nonzero(np.abs(a[nz]) >= np.abs(a[by[M - 1]]) * BAND))
        k = more if more <= M + SLACK else M
    keep = np.sort(by[:k])
    return r[keep], a[keep]


def _amps(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n)
    if kind == "equal":
        return np.full(n, 0.5)
    if kind == "few values":
        return rng.integers(-3, 4, n) * 0.25
    if kind == "near ties":  # within the band of one another
        return 1.0 + rng.integers(0, 50, n) * 2.0 ** -50
    return np.where(rng.random(n) < 0.5, np.inf, 2.0 ** rng.uniform(-1074, 1000, n))  # "extremes"


@pytest.mark.parametrize("n", [1, 1023, 16383, 16384, 16385, 300001, (4 << 20) - 1, (4 << 20) + 1])
@pytest.mark.parametrize("kind", ["normal", "equal", "few values", "near ties", "extremes"])
def test_topm_is_the_sorted_cut(P, n, kind):
    rng = np.random.default_rng(n)
    r = np.sort(rng.choice(P.n_det, n, replace=False)).astype(np.int64)
    a = _amps(kind, n, rng)
    for M in sorted({0, 1, n // 3, max(0, n - 1), n, n + 5}):
        for band in (False, True):
            gr, ga = P.topm(r, a, M, tie_band=band)
            wr, wa = _expected(r, a, M, band)
            assert np.array_equal(gr.cpu().numpy(), wr), (M, band)
            assert np.array_equal(ga.cpu().numpy(), wa), (M, band)
