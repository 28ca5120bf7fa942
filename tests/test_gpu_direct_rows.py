"""Direct summation of more targets than one row of workgroups holds: chosen targets, at the rows'
and workgroups' ends and between, against their sums in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [262_143, 262_144, 262_145, 300_001])
def test_direct_rows(n):
    """FP64 sums of n terms of either sign, in another order than numpy's pairwise one: up to n / 16 of
    them one after another, so n / 16 roundings of 1.1e-16 of the sum of their sizes at most."""
    import torch
    from paper_1406_4254_amd import etics as E
    rng = np.random.default_rng(n)
    x, y, z = rng.normal(size=(3, n))
    m = rng.uniform(0.5, 1.5, n) / n
    d = [torch.from_numpy(a).cuda() for a in (x, y, z, m)]
    pot, *acc = [t.cpu().numpy() for t in E.etics_direct_force(*d, 3)]
    acc = np.stack(acc, 1)
    X = np.stack([x, y, z], 1)
    for i in sorted({0, 63, 64, 131_071, 196_608, 262_142, n - 2, n - 1} | set(rng.integers(0, n, 24).tolist())):
        dx = X - X[i]
        r = np.sqrt((dx * dx).sum(1))
        r[i] = np.inf
        w = m / r
        tol = n / 16 * 1.2e-16
        assert abs(pot[i] + w.sum()) <= tol * w.sum(), i
        f = (w / r ** 2)[:, None] * dx
        assert np.all(np.abs(acc[i] - f.sum(0)) <= tol * np.abs(f).sum(0)), i
