"""The FP32 force of the lowest order alone (nmax = lmax = 0) at points whose squared radius
overflows FP32: the radial variable xi is NaN there, and the monopole, which has no part in
xi, is zero and not NaN (as is the Hernquist-Ostriker one's gradient on the axis, where the
direction is still known)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("basis", [0, 1])
def test_monopole_far_away(prec, basis):
    import torch
    from paper_1406_4254_amd import etics as E
    x = np.array([0.3, 1e30, 0.0, 1e25, -2.0])
    y = np.array([0.2, 0.0, 0.0, 1e25, 0.1])
    z = np.array([0.1, 0.0, 1e30, -1e25, 0.5])
    d = [torch.from_numpy(a).cuda() for a in (x, y, z)]
    A, B = torch.full((1,), 0.7, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    far, near = [1, 2, 3], [0, 4]
    for outputs in (1, 3):
        got = [None if t is None else t.cpu().numpy() for t in
               E.etics_scf_force_basis(*d, 0, 0, A, B, prec, basis, outputs)]
        ref = [None if t is None else t.cpu().numpy() for t in
               E.etics_scf_force_basis(*d, 0, 0, A, B, 0, basis, outputs)]
        assert np.all(got[0][far] == 0.0)
        np.testing.assert_allclose(got[0][near], ref[0][near], rtol=1e-5)
        if outputs == 3:
            if basis == E.ETICS_BASIS_HO:
                assert all(g[2] == 0.0 for g in got[1:])
            for g, r in zip(got[1:], ref[1:]):
                np.testing.assert_allclose(g[near], r[near], rtol=1e-4, atol=1e-6)
