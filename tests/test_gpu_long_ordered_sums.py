"""In-order sums of 65 536 and more terms, reduced over the chip block by block, equal a plain left-to-right loop bit
for bit: at the edges of the first size, of a block, of blocks of two steps, with many binade changes, ties, zeros and
sums that wander about zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [65535, 65536, 65537, 70001, 256 * 4096, 256 * 4096 + 1]


@pytest.fixture(scope="module")
def P():
    from paper_2312_01846_amd import sfci, synth

    h, g = synth.molecule_like(16, 32, 5)
    return sfci.Problem(16, 4, 4, h, g)


def _amps(kind, n, rng):
    if kind == "decaying":
        return rng.standard_normal(n) * np.exp(-np.linspace(0.0, 30.0, n))
    if kind == "growing":
        return rng.standard_normal(n) * np.exp(np.linspace(-30.0, 0.0, n))
    if kind == "ties":  # 2^53 + 1 + 1 + ...
        a = np.ones(n)
        a[:2] = 2.0 ** 26
        return a
    if kind == "zeros":  # long stretches of squares that are zero
        a = rng.standard_normal(n)
        a[5000:60000] = 1e-200
        return a
    return rng.standard_normal(n)


@pytest.mark.parametrize("kind", ["normal", "decaying", "growing", "ties", "zeros"])
@pytest.mark.parametrize("n", SIZES)
def test_norm_is_the_sequential_sum(P, kind, n):
    rng = np.random.default_rng(3)
    a = _amps(kind, n, rng)
    r = np.arange(n, dtype=np.int64)
    _, got = P.topm(r, a, n, normalise=True)
    ss = np.add.accumulate(a * a)[-1]
    assert np.array_equal(got.cpu().numpy(), a / np.sqrt(ss))


@pytest.mark.parametrize("n", [70001, 100000])
def test_energy_numerator_is_the_sequential_sum(P, n):
    rng = np.random.default_rng(4)
    r = np.sort(rng.choice(P.n_det, n, replace=False)).astype(np.int64)
    a = rng.standard_normal(n)
    e, _, _ = P.energy_gradients(r, a, deterministic=True, want_grad=False)
    yr, ya, _ = P.sigma(r, a, M=None, deterministic=True)
    D = np.zeros(P.n_det)
    D[yr.cpu().numpy()] = ya.cpu().numpy()
    num = np.add.accumulate(a * D[r])[-1]
    assert e == num / np.add.accumulate(a * a)[-1]
