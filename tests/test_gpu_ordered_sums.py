"""In-order sums (the norm of a truncation, the energy's numerator in deterministic mode) equal a plain
left-to-right loop bit for bit: binade changes, ties, zeros and extreme magnitudes, at the edges of the
kernel's lanes (8 terms), chunks (512) and steps (4096)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 64, 65, 511, 513, 4095, 4096, 4097, 20011]


@pytest.fixture(scope="module")
def P():
    from paper_2312_01846_amd import sfci, synth

    h, g = synth.molecule_like(12, 24, 5)
    return sfci.Problem(12, 4, 4, h, g)


def _amps(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n)
    if kind == "decaying":
        return rng.standard_normal(n) * np.exp(-np.linspace(0.0, 30.0, n))
    if kind == "wide":
        return np.exp(4.0 * rng.standard_normal(n))
    if kind == "integers":
        return rng.integers(1, 9, n).astype(np.float64)
    if kind == "ties":  # 2^53 + 1 + 1 + ...: every addition is half way between two doubles
        a = np.ones(n)
        a[:2] = 2.0 ** 26
        return a
    if kind == "odd ties":  # an odd multiple of the unit first, so that ties round up
        a = np.ones(n)
        a[:3] = [2.0 ** 26, 2.0 ** 26, 2.0 ** 0.5][:n]
        return a
    if kind == "tiny":  # squares in the subnormal range and below
        return 2.0 ** rng.uniform(-545.0, -530.0, n)
    return 2.0 ** rng.uniform(-500.0, 400.0, n)  # "huge range"


@pytest.mark.parametrize("kind", ["normal", "decaying", "wide", "integers", "ties", "odd ties", "tiny", "huge range"])
def test_norm_of_truncation_is_the_sequential_sum(P, kind):
    rng = np.random.default_rng(3)
    for n in SIZES:
        a = _amps(kind, n, rng)
        r = np.sort(rng.choice(P.n_det, n, replace=False)).astype(np.int64)
        _, got = P.topm(r, a, n, normalise=True)
        ss = np.add.accumulate(a * a)[-1]
        want = a / np.sqrt(ss) if ss > 0.0 else a
        assert np.array_equal(got.cpu().numpy(), want), (kind, n)


def test_energy_numerator_is_the_sequential_sum(P):
    rng = np.random.default_rng(4)
    for n in SIZES[1:]:
        r = np.sort(rng.choice(P.n_det, n, replace=False)).astype(np.int64)
        a = rng.standard_normal(n)
        e, _, _ = P.energy_gradients(r, a, deterministic=True, want_grad=False)
        yr, ya, _ = P.sigma(r, a, M=None, deterministic=True)
        yr, ya = yr.cpu().numpy(), ya.cpu().numpy()
        at = np.minimum(np.searchsorted(yr, r), yr.size - 1)
        y = np.where(yr[at] == r, ya[at], 0.0)
        assert e == np.add.accumulate(a * y)[-1] / np.add.accumulate(a * a)[-1], n
