"""The FP32 force pass on the matrix cores, at the edges of its layout: odd and even nmax
(pairs of orders), every lmax bucket with lmax at and below it (one or two coefficient
registers per pair), partly filled wavefronts, and the three output modes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1406_4254_amd import accuracy as acc  # noqa: E402
from paper_1406_4254_amd import workloads as W  # noqa: E402

MIXED = 1


def dev(*arrs):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in arrs]


@pytest.mark.parametrize("n", [1, 63, 65, 257])
@pytest.mark.parametrize("nmax,lmax", [(0, 0), (1, 0), (1, 1), (2, 2), (3, 3), (4, 5), (1, 7), (6, 8), (9, 9), (2, 11),
                                       (11, 12), (19, 13), (20, 14)])
def test_force_quads(orc, nmax, lmax, n):
    """FP32 sums of up to (nmax+1)(lmax+1)^2 <= 4725 products of either sign: rounding of
    about 6e-8 sqrt(4725) = 4e-6 of a particle's force or potential; 25 times that."""
    from paper_1406_4254_amd import etics as E
    q = W.make_config(2, 4000)
    A, B = orc.scf_coeffs(q.x, q.y, q.z, q.m, nmax, lmax)
    x, y, z = q.x[:n], q.y[:n], q.z[:n]
    rp, rx, ry, rz = orc.scf_force(x, y, z, nmax, lmax, A, B)
    d, c = dev(x, y, z), dev(A, B)
    for outputs in (1, 2, 3):
        pot, ax, ay, az = [None if t is None else t.cpu().numpy()
                           for t in E.etics_scf_force(*d, nmax, lmax, *c, MIXED, outputs)]
        if outputs & 1:
            assert np.max(acc.pot_rel_err(pot, rp)) < 1e-4
        if outputs & 2:
            assert np.max(acc.force_rel_err(ax, ay, az, rx, ry, rz)) < 1e-4


@pytest.mark.parametrize("n,nmax,lmax", [(399_999, 3, 7), (400_000, 3, 7), (400_000, 2, 6)])
def test_fp64_potential_sources(orc, n, nmax, lmax):
    """FP64 potential alone on both sides of the size where the coefficients become scalar
    operands, and below lmax 7 where they never do; FP64 rounding of sums of at most 256
    products against the oracle (the bound of the other FP64 potential tests)."""
    from paper_1406_4254_amd import etics as E
    p = W.make_config(2, n)
    A, B = orc.scf_coeffs(p.x[:4000], p.y[:4000], p.z[:4000], p.m[:4000], nmax, lmax)
    pot = E.etics_scf_force(*dev(p.x, p.y, p.z), nmax, lmax, *dev(A, B), 0, 1)[0].cpu().numpy()
    rp = orc.scf_force(p.x, p.y, p.z, nmax, lmax, A, B)[0]
    assert np.max(acc.pot_rel_err(pot, rp)) < 1e-13
