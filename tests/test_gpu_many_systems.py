"""The FP32 preparation of more coefficients than one trip of its grid covers: forces of many
small systems at the largest cutoffs against the single-system call on the same coefficients."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_many_systems_largest_cutoffs():
    import torch
    from paper_1406_4254_amd import etics as E
    nsys, per, nmax, lmax = 2000, 3, 20, 14  # 2.1 10^7 prepared values; a trip is 1.7 10^7
    rng = np.random.default_rng(2)
    n = nsys * per
    x = rng.normal(size=(3, n))
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in x]
    m = torch.full((n,), 1.0 / per, dtype=torch.float64, device="cuda")
    off = torch.arange(0, n + 1, per, dtype=torch.int64, device="cuda")
    ws = E.workspace(E.etics_batched_workspace_size(n, nsys, nmax, lmax, E.ETICS_MIXED_FP64ACC), "cuda")
    A, B = E.etics_scf_coeffs_batched(*d, m, off, nmax, lmax, ws=ws)
    got = torch.stack(E.etics_scf_force_batched(*d, off, nmax, lmax, A, B, ws=ws))
    K = E.etics_coeff_count(nmax, lmax)
    for s in (0, 1, 1597, 1598, 1599, 1998, 1999):
        a, b = A.view(nsys, K)[s].contiguous(), B.view(nsys, K)[s].contiguous()
        i = slice(s * per, (s + 1) * per)
        ref = torch.stack(E.etics_scf_force(*[t[i].contiguous() for t in d], nmax, lmax, a, b))
        # the same arithmetic in both kernels
        torch.testing.assert_close(got[:, i], ref, rtol=1e-5, atol=1e-5 * float(ref.abs().max()))
