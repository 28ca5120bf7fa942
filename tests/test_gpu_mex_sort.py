"""The particle order of MEX on both sides of every line between its sorts, with equal keys,
and with inputs that the sample sort's samples miss, against an argsort of the keys.

The potential of the monopole (lmax = 0) tells the order: with masses 2^-(index mod 40) a
pair in the wrong order, or a particle counted twice, changes the sums far beyond rounding.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def monopole(x, y, z, m):
    """-(M(before) / r + sum of m/r after), particles ordered by (key, index)."""
    key = (x * x + y * y) + z * z
    o = np.argsort(key, kind="stable")
    r, mo = np.sqrt(key[o]), m[o].astype(np.longdouble)
    inner = np.concatenate([[0], np.cumsum(mo)[:-1]])
    w = mo / r
    outer = np.concatenate([np.cumsum(w[::-1])[::-1][1:], [0]])
    pot = np.empty(len(x))
    pot[o] = -(inner / r + outer)
    return pot


def check(x, y, z):
    import torch
    from paper_1406_4254_amd import etics as E
    n = len(x)
    m = 2.0 ** -(np.arange(n) % 40)
    d = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in (x, y, z, m)]
    pot = E.etics_mex_force(*d, 0, 0, 1)[0].cpu().numpy()
    ref = monopole(x, y, z, m)
    # FP64 sums of up to 10^6 positive terms in trees: a few roundings each
    np.testing.assert_allclose(pot, ref, rtol=1e-13)


def cloud(n, seed):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal((3, n))
    return v / np.linalg.norm(v, axis=0) * rng.random(n) ** (1 / 3) * 3


@pytest.mark.parametrize("n", [1, 2, 17, 8191, 8192, 8193, 8200, 65_537, 1_048_576, 1_048_577])
def test_sort_sizes(n):
    check(*cloud(n, n))


@pytest.mark.parametrize("n", [5000, 50_000, 300_000])
@pytest.mark.parametrize("kind", ["lattice", "shell", "sorted", "reversed", "wide"])
def test_sort_inputs(n, kind):
    """Many equal keys (integer positions; a shell, whose keys differ in the last bits), the
    keys already in order or reversed, and radii over 60 decades."""
    rng = np.random.default_rng(n)
    if kind == "lattice":
        x, y, z = rng.integers(-9, 10, (3, n)).astype(float)
        x[(x == 0) & (y == 0) & (z == 0)] = 1.0
    elif kind == "shell":
        v = rng.standard_normal((3, n))
        x, y, z = v / np.linalg.norm(v, axis=0)
    elif kind == "wide":
        x, y, z = cloud(n, 1) * 10.0 ** rng.uniform(-30, 30, n)
    else:
        x, y, z = cloud(n, 2)
        o = np.argsort(x * x + y * y + z * z)
        o = o[::-1] if kind == "reversed" else o
        x, y, z = x[o], y[o], z[o]
    check(x, y, z)


def test_sort_bucket_beyond_lds():
    """Particles where the samples are taken lie further in than all the others, so the last
    bucket holds nearly everything and is sorted through memory."""
    n, samples = 100_000, 4096
    s = np.arange(samples, dtype=np.uint64)
    a, b = s * n // samples, (s + 1) * n // samples
    h = (s * 2654435761) & 0xFFFFFFFF
    h ^= h >> np.uint64(15)
    at = a + ((h * (b - a)) >> np.uint64(32))
    x, y, z = cloud(n, 3)
    r = np.sqrt(x * x + y * y + z * z)
    scale = (5.0 + np.random.default_rng(4).random(n)) / r
    scale[at] = 0.5 / r[at] * np.random.default_rng(5).random(samples)
    check(x * scale, y * scale, z * scale)
