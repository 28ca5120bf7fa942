"""The particle order of MEX where keys are equal or differ in their last bits, in every one of
its sorts, told by the monopole's acceleration: -(mass before) / r^2 along r, which steps by a
particle's own mass where two particles change places (the potential has no such step: at equal
radius a particle counts the same inside and outside)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def masses(n):
    return 1.0 + np.arange(n) % 7


def mass_before(x, y, z, m):
    """Of the particles ordered by (key, index), at each particle."""
    o = np.argsort((x * x + y * y) + z * z, kind="stable")
    before = np.empty(len(x))
    before[o] = np.concatenate([[0.0], np.cumsum(m[o])[:-1]])
    return before


def check(x, y, z):
    import torch
    from paper_1406_4254_amd import etics as E
    m = masses(len(x))
    d = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in (x, y, z, m)]
    _, ax, ay, az = [None if t is None else t.cpu().numpy() for t in E.etics_mex_force(*d, 0, E.ETICS_FP64, 2)]
    got = -(ax * x + ay * y + az * z) * np.sqrt((x * x + y * y) + z * z)
    # the lightest particle is 1; the sums reach 5e6, whose FP64 rounding is far below
    np.testing.assert_allclose(got, mass_before(x, y, z, m), rtol=0, atol=0.1)


def lattice(rng, n):
    p = rng.integers(-9, 10, (3, n)).astype(float)
    p[0, (p == 0).all(axis=0)] = 1.0
    return p


def shell(rng, n):
    v = rng.standard_normal((3, n))
    return v / np.linalg.norm(v, axis=0)


def inputs(kind, n):
    rng = np.random.default_rng(n)
    if kind == "lattice":
        return lattice(rng, n)
    if kind == "shell":
        return shell(rng, n)
    if kind == "one":  # a single key
        return np.repeat([[0.5], [-0.25], [1.0]], n, axis=1)
    p = lattice(rng, n)  # sorted: the keys in order already, or reversed, with all their ties
    o = np.argsort((p * p).sum(0), kind="stable")
    return p[:, o[::-1] if kind == "reversed" else o]


# the rank count, the sample sort and the radix sort
@pytest.mark.parametrize("n", [5000, 8192, 8193, 50_000, 300_000, 1_048_576, 1_048_577, 1_200_000])
@pytest.mark.parametrize("kind", ["lattice", "shell", "one", "sorted", "reversed"])
def test_order_of_ties(kind, n):
    check(*inputs(kind, n))


@pytest.mark.parametrize("kind", ["lattice", "shell"])
def test_order_of_ties_beyond_lds(kind):
    """Particles where the sample sort takes its samples lie further in than all the others, so
    the last bucket holds nearly everything and goes through memory, ties and all."""
    n, samples = 100_000, 4096
    s = np.arange(samples, dtype=np.uint64)
    a, b = s * n // samples, (s + 1) * n // samples
    h = (s * 2654435761) & 0xFFFFFFFF
    h ^= h >> np.uint64(15)
    at = (a + ((h * (b - a)) >> np.uint64(32))).astype(np.int64)
    x, y, z = inputs(kind, n)
    rng = np.random.default_rng(6)
    x[at], y[at], z[at] = shell(rng, samples) * 0.5 * rng.random(samples)
    check(x, y, z)


def test_ties_change_the_expected_values():
    """What the test holds on to: another order of equal keys moves the expected values by more than
    the tolerance."""
    for kind in ("lattice", "one"):
        x, y, z = inputs(kind, 5000)
        m = masses(5000)
        ref = mass_before(x, y, z, m)
        back = mass_before(x[::-1], y[::-1], z[::-1], m[::-1])[::-1]  # ties in reversed order
        assert np.max(np.abs(ref - back)) >= 1.0
